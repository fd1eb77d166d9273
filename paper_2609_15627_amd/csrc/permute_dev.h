// The 16-wave placement of the expert sorter (see permute.hip), for kernels that
// sort in one workgroup of 1024 threads.
#pragma once

#include "moe_dev.h"

namespace moe {

constexpr int kChunk = 1024;   // assignments per chunk
constexpr int kSmallNE = 512;  // experts whose per-wave counts fit LDS

// Wave-level part of the 16-wave placement: assignment a of this lane (a < A
// taken), its expert e (ok: a valid id) and its rank among the wave's
// earlier lanes with the same expert; the group's highest lane records the
// group size in cnt[w * NE + e] (cnt zeroed beforehand, a barrier after).
__device__ __forceinline__ void wave_rank16(const int32_t* ids, int a, int A, int NE,
                                            int nbits, int32_t* cnt, int* e_out, bool* ok_out,
                                            int* rank_out) {
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int e = a < A ? ids[a] : -1;
  const bool ok = (unsigned)e < (unsigned)NE;
  uint64_t peers = __ballot(ok);
  for (int b = 0; b < nbits; ++b) {
    const bool bit = ok && ((e >> b) & 1);
    const uint64_t m = __ballot(bit);
    peers &= bit ? m : ~m;
  }
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
  const int rank = __popcll(peers & lt);
  __syncthreads();  // cnt was zeroed by other threads
  if (ok && (peers >> lane) == 1ull) cnt[w * NE + e] = rank + 1;
  *e_out = e;
  *ok_out = ok;
  *rank_out = rank;
}

// Exclusive prefix of the 16 per-wave counts of expert threadIdx.x (in
// place); returns the expert's total. Call after a barrier.
__device__ __forceinline__ int prefix_waves16(int32_t* cnt, int NE) {
  int c = 0;
  if ((int)threadIdx.x < NE) {
    int n[16];  // all reads first: one LDS round trip instead of sixteen
#pragma unroll
    for (int v = 0; v < 16; ++v) n[v] = cnt[v * NE + threadIdx.x];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      cnt[v * NE + threadIdx.x] = c;
      c += n[v];
    }
  }
  return c;
}

// Places chunk `chunk` of the assignments by a workgroup of 1024 threads; thread
// e < NE gives the chunk's first slot of its expert; sh: 17 NE ints of LDS.
__device__ __forceinline__ void perm_place_chunk(const int32_t* __restrict__ ids, int chunk, int A,
                                                 int NE, int nbits, int first, int32_t* sh,
                                                 int32_t* __restrict__ sorted,
                                                 int32_t* __restrict__ pos) {
  int32_t* cnt = sh;             // [16][NE]
  int32_t* base = sh + 16 * NE;  // [NE]
  for (int i = threadIdx.x; i < 16 * NE; i += blockDim.x) cnt[i] = 0;
  if ((int)threadIdx.x < NE) base[threadIdx.x] = first;
  const int a = chunk * kChunk + (int)threadIdx.x;
  int e, rank;
  bool ok;
  wave_rank16(ids, a, A, NE, nbits, cnt, &e, &ok, &rank);
  __syncthreads();
  prefix_waves16(cnt, NE);
  __syncthreads();
  if (ok) {
    const int dest = base[e] + cnt[(threadIdx.x / kWave) * NE + e] + rank;
    sorted[dest] = a;
    pos[a] = dest;
  }
}

// The whole sort of A <= kChunk assignments over NE <= kSmallNE experts by one
// workgroup; sh: 17 NE ints of LDS. Thread e < NE gets its expert's count and
// first slot.
__device__ __forceinline__ void perm_place16(const int32_t* ids, int A, int NE, int nbits,
                                             int32_t* sh, int32_t* __restrict__ counts,
                                             int32_t* __restrict__ offsets,
                                             int32_t* __restrict__ sorted,
                                             int32_t* __restrict__ pos, int* count, int* first) {
  int32_t* cnt = sh;            // [16][NE]: per-wave counts, then their prefix over waves
  int32_t* off = sh + 16 * NE;  // [NE]: expert offsets
  for (int i = threadIdx.x; i < 16 * NE; i += blockDim.x) cnt[i] = 0;
  int e, rank;
  bool ok;
  wave_rank16(ids, (int)threadIdx.x, A, NE, nbits, cnt, &e, &ok, &rank);
  __syncthreads();
  const int c = prefix_waves16(cnt, NE);
  int total;
  const int p0 = block_exclusive_scan_1024(c, &total);
  if ((int)threadIdx.x < NE) {
    counts[threadIdx.x] = c;
    offsets[threadIdx.x] = p0;
    off[threadIdx.x] = p0;
  }
  if (threadIdx.x == 0) offsets[NE] = total;
  __syncthreads();
  if (ok) {
    const int dest = off[e] + cnt[(threadIdx.x / kWave) * NE + e] + rank;
    sorted[dest] = threadIdx.x;
    pos[threadIdx.x] = dest;
  }
  *count = c;
  *first = p0;
}

}  // namespace moe
