// The steps before the expert GEMMs as one launch, for small batches: routing
// (few tokens), the expert sort, the row-tile lists and the quantisation of x.
//
// At decode each of these steps is a kernel of a few microseconds that waits
// mostly for its own start and for the round trips of its small inputs, and the
// layer waits for all of them in a row (one token: routing 6.1, sort 3.6,
// quantisation and tile lists 6.4 us, and a gap at each border, against 27 us for
// both expert GEMMs). Block 0 (16 waves) routes, sorts and lists; the other
// blocks quantise x meanwhile. The sort's counts and first slots are in
// registers when the tile list needs them, so that takes one scan.
// Routing joins while every wave has at most one token (kFrontTokens): with
// more, one CU's vector units take longer over the arg-max rounds than a launch
// of its own that spreads the tokens over many CUs.
#include "gemm_common.h"
#include "moe_launch.h"
#include "permute_dev.h"
#include "quant_dev.h"
#include "route_dev.h"
#include "tiles_dev.h"

namespace moe {

// Row tiles of BM rows from each expert's count c and first row r0 (thread e
// holds expert e).
__device__ __forceinline__ void front_tiles(const TileArgs& t, int BM, int NE, int c, int r0) {
  const int m = (int)threadIdx.x < NE ? (c + BM - 1) / BM : 0;
  int total;
  const int ts = block_exclusive_scan_1024(m, &total);
  int4* tiles = const_cast<int4*>(t.tiles);
  for (int j = 0; j < m; ++j)
    tiles[ts + j] = make_int4((int)threadIdx.x, r0 + j * BM, min(BM, c - j * BM), m);
  if (threadIdx.x == 0) *const_cast<int*>(t.ntiles) = total;
}

// Logits a lane group of these kernels holds; a router may have more columns than
// there are experts (an id past the last one is left out of the sort).
constexpr int kFrontE = 8 * kWave;

// EPL: experts per lane of the routing, 0: the ids are given.
template <int FMT, int EPL>
__global__ __launch_bounds__(1024) void front_kernel(FrontArgs a) {
  if (blockIdx.x > 0) {
    if constexpr (FMT >= 0) {
      const long b = (long)(blockIdx.x - 1) * 1024 + threadIdx.x;
      if (b < a.nblk) quant_block<FMT, true>(a.x, b, a.codes, a.scales);
    }
    return;
  }
  extern __shared__ int32_t sh[];
  const int kt = a.k + a.n_shared;
  const int32_t* ids = a.ids;
  if constexpr (EPL > 0) {
    int32_t* sids = sh + 17 * a.NE;  // [A]
    const int t = threadIdx.x / kWave;
    if (t < a.T)
      route_plain_token<EPL>(a.logits + (size_t)t * a.E, a.E, a.k, a.n_shared, a.ids + t * kt,
                             a.w + t * kt, threadIdx.x % kWave, sids + t * kt);
    ids = sids;
    __syncthreads();
  }
  int c, r0;
  perm_place16(ids, a.T * kt, a.NE, a.nbits, sh, a.counts, a.offsets, a.sorted, a.pos, &c, &r0);
  front_tiles(a.t1, a.BM1, a.NE, c, r0);
  if (a.BM2 != a.BM1) front_tiles(a.t2, a.BM2, a.NE, c, r0);
}

template <int FMT>
static void launch_front_fmt(const FrontArgs& a, hipStream_t s) {
  const int kt = a.k + a.n_shared;
  const dim3 grid(1 + (int)((a.nblk + 1023) / 1024)), block(1024);
  const bool route = a.logits != nullptr;
  const size_t lds = ((size_t)17 * a.NE + (route ? a.T * kt : 0)) * sizeof(int32_t);
  const int epl = route ? (a.E + kWave - 1) / kWave : 0;
  if (epl == 0) hipLaunchKernelGGL((front_kernel<FMT, 0>), grid, block, lds, s, a);
  else if (epl == 1) hipLaunchKernelGGL((front_kernel<FMT, 1>), grid, block, lds, s, a);
  else if (epl == 2) hipLaunchKernelGGL((front_kernel<FMT, 2>), grid, block, lds, s, a);
  else if (epl <= 4) hipLaunchKernelGGL((front_kernel<FMT, 4>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((front_kernel<FMT, 8>), grid, block, lds, s, a);
}

bool front_sizes_ok(int T, int NE, int k_total) {
  return T > 0 && (long)T * k_total <= kChunk && NE <= kSmallNE;
}

bool front_routes(int T, int E) { return T <= kFrontTokens && E <= kFrontE; }

hipError_t launch_front(const FrontArgs& a0, hipStream_t s) {
  FrontArgs a = a0;
  a.nbits = 0;
  while ((1 << a.nbits) < a.NE) ++a.nbits;
  if (a.fmt == kFmtBf16) launch_front_fmt<-1>(a, s);
  else if (a.fmt == 0) launch_front_fmt<0>(a, s);
  else if (a.fmt == 2) launch_front_fmt<2>(a, s);
  else launch_front_fmt<4>(a, s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Larger batches: three launches instead of five or six.
//  1. routing and the quantisation of x side by side (routing is bound by its
//     arg-max latency, the quantisation by memory);
//  2. the chunk histograms of the sort (perm_hist);
//  3. the scatter, whose workgroups add up the histograms of the chunks before
//     theirs themselves (up to kFrontChunks chunks; a scan kernel of its own took
//     4.9 us and a gap), beside one workgroup per row-tile list, which needs only
//     the counts.
// 4096 tokens, top-8 of 256, H = 4096: 42 us of kernels in five launches before.
// ---------------------------------------------------------------------------
constexpr int kFrontChunks = 96;

template <int FMT, int EPL>
__global__ __launch_bounds__(256) void route_quant_kernel(FrontArgs a, int nrb) {
  if ((int)blockIdx.x < nrb) {
    const int t = (int)blockIdx.x * 4 + (int)threadIdx.x / kWave;
    if (t >= a.T) return;
    const int kt = a.k + a.n_shared;
    route_plain_token<EPL>(a.logits + (size_t)t * a.E, a.E, a.k, a.n_shared,
                           a.ids + (size_t)t * kt, a.w + (size_t)t * kt, threadIdx.x % kWave);
    return;
  }
  if constexpr (FMT >= 0) {
    const long b = (long)(blockIdx.x - nrb) * 256 + threadIdx.x;
    if (b < a.nblk) quant_block<FMT, true>(a.x, b, a.codes, a.scales);
  }
}

__global__ __launch_bounds__(1024) void sort_tiles_kernel(FrontArgs a, int A, int nchunks) {
  extern __shared__ int32_t sh[];
  const int NE = a.NE, e = (int)threadIdx.x, chunk = (int)blockIdx.x;
  int before = 0, c = 0;  // assignments of expert e in earlier chunks, and in all
  if (e < NE) {
    for (int i = 0; i < nchunks; i += 24) {  // 24 loads in flight a thread
      int n[24];
#pragma unroll
      for (int j = 0; j < 24; ++j) n[j] = a.hist[(size_t)min(i + j, nchunks - 1) * NE + e];
#pragma unroll
      for (int j = 0; j < 24; ++j) {
        if (i + j < nchunks) c += n[j];
        if (i + j < min(chunk, nchunks)) before += n[j];
      }
    }
  }
  int total;
  const int off = block_exclusive_scan_1024(c, &total);
  if (chunk < nchunks) {
    if (chunk == 0) {
      if (e < NE) {
        a.counts[e] = c;
        a.offsets[e] = off;
      }
      if (e == 0) a.offsets[NE] = total;
    }
    perm_place_chunk(a.ids, chunk, A, NE, a.nbits, off + before, sh, a.sorted, a.pos);
    return;
  }
  // a tile list
  if (e < NE) sh[e] = off;
  if (e == 0) sh[NE] = total;
  __syncthreads();
  const bool first = chunk == nchunks;
  const TileArgs& t = first ? a.t1 : a.t2;
  build_tiles(sh, NE, first ? a.BM1 : a.BM2, const_cast<int4*>(t.tiles),
              const_cast<int*>(t.ntiles), const_cast<int4*>(t.chunks), const_cast<int*>(t.nchunks),
              t.queue, sh + NE + 1);
}

template <int FMT>
static void launch_route_quant(const FrontArgs& a, hipStream_t s) {
  const int nrb = (a.T + 3) / 4;
  const dim3 grid(nrb + (int)((a.nblk + 255) / 256)), block(256);
  const int epl = (a.E + kWave - 1) / kWave;
  if (epl <= 1) hipLaunchKernelGGL((route_quant_kernel<FMT, 1>), grid, block, 0, s, a, nrb);
  else if (epl == 2) hipLaunchKernelGGL((route_quant_kernel<FMT, 2>), grid, block, 0, s, a, nrb);
  else if (epl <= 4) hipLaunchKernelGGL((route_quant_kernel<FMT, 4>), grid, block, 0, s, a, nrb);
  else hipLaunchKernelGGL((route_quant_kernel<FMT, 8>), grid, block, 0, s, a, nrb);
}

bool front_large_sizes_ok(int T, int NE, int k_total, int E) {
  const long A = (long)T * k_total;
  return E <= kFrontE && A > kChunk && A <= (long)kFrontChunks * kChunk && NE <= kSmallNE;
}

hipError_t launch_front_large(const FrontArgs& a0, hipStream_t s) {
  FrontArgs a = a0;
  a.nbits = 0;
  while ((1 << a.nbits) < a.NE) ++a.nbits;
  if (a.fmt == kFmtBf16) launch_route_quant<-1>(a, s);
  else if (a.fmt == 0) launch_route_quant<0>(a, s);
  else if (a.fmt == 2) launch_route_quant<2>(a, s);
  else launch_route_quant<4>(a, s);
  const int A = a.T * (a.k + a.n_shared), nchunks = (A + kChunk - 1) / kChunk;
  const hipError_t e = launch_perm_hist(a.ids, A, a.NE, a.hist, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sort_tiles_kernel, dim3(nchunks + (a.BM2 == a.BM1 ? 1 : 2)), dim3(1024),
                     (size_t)17 * a.NE * sizeof(int32_t), s, a, A, nchunks);
  return hipGetLastError();
}

}  // namespace moe
