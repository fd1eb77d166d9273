// Top-k selection and softmax weights of one token by one wave (see route.hip).
#pragma once

#include "moe_dev.h"

namespace moe {

// EPL = experts held per lane (ceil(E / 64) rounded up to a power of two); the
// token's E logits at row, its k + n_shared ids and weights to id_row and w_row
// (and the ids to lds_ids, if not null).
template <int EPL>
__device__ __forceinline__ void route_plain_token(const float* __restrict__ row, int E, int k,
                                                  int n_shared, int32_t* __restrict__ id_row,
                                                  float* __restrict__ w_row, int lane,
                                                  int32_t* lds_ids = nullptr) {
  float v[EPL];
  bool live[EPL];
#pragma unroll
  for (int j = 0; j < EPL; ++j) {
    const int e = lane + kWave * j;
    live[j] = e < E;
    float x = live[j] ? row[e] : -INFINITY;
    v[j] = (x != x) ? -INFINITY : x;  // NaN reads as -inf
  }
  float my_val = 0.0f;
  int my_id = 0;
  for (int r = 0; r < k; ++r) {
    float bv = -INFINITY;
    int bi = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const int e = lane + kWave * j;
      if (live[j] && (v[j] > bv || (v[j] == bv && e < bi))) {
        bv = v[j];
        bi = e;
      }
    }
    wave_argmax(bv, bi);
    // every lane now holds the same (bv, bi); retire the pick
#pragma unroll
    for (int j = 0; j < EPL; ++j)
      if (lane + kWave * j == bi) live[j] = false;
    if (lane == r) {
      my_val = bv;
      my_id = bi;
    }
  }
  const float l0 = lane_value(my_val, 0);
  const float ex = lane < k ? expf(my_val - l0) : 0.0f;
  float den = 0.0f;
  for (int j = 0; j < k; ++j) den += lane_value(ex, j);
  if (lane < k) {
    id_row[lane] = my_id;
    w_row[lane] = ex / den;
    if (lds_ids) lds_ids[lane] = my_id;
  } else if (lane == k && n_shared) {
    id_row[lane] = E;
    w_row[lane] = 1.0f;
    if (lds_ids) lds_ids[lane] = E;
  }
}

}  // namespace moe
