// The row-tile lists of the grouped GEMM's geometries, built by one workgroup of
// 1024 threads.
#pragma once

#include "gemm_common.h"

namespace moe {

// ---------------------------------------------------------------------------
// Tile list: expert e with c rows gets ceil(c / BM) row tiles. One block of
// 1024 threads: tile counts, exclusive scan, then every thread fills tiles
// i = tid, tid + 1024, ... by binary search over the per-expert tile starts.
//
// The work queue of the persistent tiled kernels starts at zero here; each
// of their launches leaves it at zero when it ends.
//
// Chunk list (the tiled geometry launches C row tiles at a time, so that
// they share their weight rows in L2). C = 2 (256-row tiles): an expert's
// tiles pair up among themselves, so its weights are never split across two
// chunks; the odd tile left over by an expert pairs with the next expert's
// leftover. Chunk order: all within-expert pairs (expert order), then the
// leftover pairs. C = 4 (128-row tiles): an expert's tiles in groups of
// four, the last group of each expert padded with empty places (-1).
// offsets: global or LDS; start: NE + 1 ints of LDS.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void build_tiles(const int32_t* offsets, int NE, int BM,
                                            int4* __restrict__ tiles, int* __restrict__ ntiles,
                                            int4* __restrict__ chunks, int* __restrict__ nchunks,
                                            int* __restrict__ queue, int* start) {
  const int C = BM == 128 ? 4 : 2;  // row tiles per chunk
  int m[2], tot[3][2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = threadIdx.x + 1024 * q;
    m[q] = e < NE ? (offsets[e + 1] - offsets[e] + BM - 1) / BM : 0;
  }
  // exclusive prefix of: tiles, within-expert chunks (pairs, or groups of
  // four with the last one padded), leftover singles (C = 2 only)
  int p0[3], p1[3];
  auto per_expert = [&](int k, int mv) {
    if (k == 0) return mv;
    if (C == 4) return k == 1 ? (mv + 3) / 4 : 0;
    return k == 1 ? mv / 2 : mv % 2;
  };
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int v0 = per_expert(k, m[0]);
    const int v1 = per_expert(k, m[1]);
    p0[k] = block_exclusive_scan_1024(v0, &tot[k][0]);
    p1[k] = block_exclusive_scan_1024(v1, &tot[k][1]) + tot[k][0];
  }
  const int total = tot[0][0] + tot[0][1];
  const int pairs = tot[1][0] + tot[1][1];
  const int singles = tot[2][0] + tot[2][1];
  if (threadIdx.x < NE) start[threadIdx.x] = p0[0];
  if (threadIdx.x + 1024 < NE) start[threadIdx.x + 1024] = p1[0];
  if (threadIdx.x < kQueueInts) queue[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    start[NE] = total;
    *ntiles = total;
    *nchunks = pairs + (singles + 1) / 2;
    if (singles & 1) chunks[pairs + singles / 2].y = -1;  // (C = 2; C = 4 has no singles)
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = threadIdx.x + 1024 * q;
    if (e >= NE) continue;
    const int ts = q ? p1[0] : p0[0], pr = q ? p1[1] : p0[1], sg = q ? p1[2] : p0[2];
    if (C == 4) {
      const int mq = m[q];
      for (int j = 0; j < (mq + 3) / 4; ++j) {
        const int b = 4 * j;
        chunks[pr + j] = make_int4(ts + b, b + 1 < mq ? ts + b + 1 : -1, b + 2 < mq ? ts + b + 2 : -1,
                                   b + 3 < mq ? ts + b + 3 : -1);
      }
      continue;
    }
    for (int j = 0; j < m[q] / 2; ++j) chunks[pr + j] = make_int4(ts + 2 * j, ts + 2 * j + 1, -1, -1);
    if (m[q] & 1) {
      int* c = reinterpret_cast<int*>(&chunks[pairs + sg / 2]);
      c[sg & 1] = ts + m[q] - 1;
      if ((sg & 1) == 0) c[2] = c[3] = -1;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < total; i += 1024) {
    int lo = 0, hi = NE;  // find e with start[e] <= i < start[e + 1]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (start[mid] <= i) lo = mid; else hi = mid;
    }
    const int j = i - start[lo];
    const int r0 = offsets[lo] + j * BM;
    tiles[i] = make_int4(lo, r0, min(BM, offsets[lo + 1] - r0), start[lo + 1] - start[lo]);
  }
}

}  // namespace moe
