// Top-k selection of one token row held in registers: shared by the routing kernel and by the gate-network kernel
// that routes straight from its partial sums.
#pragma once
#include "common.h"

namespace moe355 {

// Order-preserving map from finite fp32 to uint32 (larger float <=> larger key); -0 and +0 map to the same
// key so that they tie, as they do under a float comparison.  Key 0 is never produced by a finite value and
// marks an expert that has already been picked.
__device__ __forceinline__ uint32_t ordered_key(float v) {
  const uint32_t b = __float_as_uint(v + 0.0f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Maximum over the wave, returned in every lane: butterfly inside the rows of 16 lanes with data-parallel
// primitives (lane ^ 1, lane ^ 2, mirrored halves, mirrored row), then the four row results are combined.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  auto step = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // row_half_mirror
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row_mirror
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return step(step(a, b), step(c, d));
}

// The value behind a key (-0 comes back as +0).
__device__ __forceinline__ float key_value(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? k ^ 0x80000000u : ~k); }

// A token row in registers, lane l owning experts [l * PER, l * PER + PER), from which the largest is picked again and
// again (key = ordered_key(value), 0 for experts past E).  Every lane sorts its run once (adjacent exchanges on strict
// comparison: equal keys keep the lower index in front), so that a pick only compares the lanes' heads.  Ties across lanes
// go to the lowest lane.  (Scanning the run and clearing a key for every pick was two thirds of the routing kernel's
// instructions, and those, not the logits, are what it takes its time for.)
template <int PER>
struct RowPicker {
  uint32_t key[PER];
  int idx[PER];
  __device__ __forceinline__ void sort() {
#pragma unroll
    for (int i = 0; i < PER; ++i) idx[i] = i;
#pragma unroll
    for (int n = PER - 1; n > 0; --n)
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const bool up = key[i + 1] > key[i];
        const uint32_t k = key[i];
        const int x = idx[i];
        key[i] = up ? key[i + 1] : k;
        idx[i] = up ? idx[i + 1] : x;
        key[i + 1] = up ? k : key[i + 1];
        idx[i + 1] = up ? x : idx[i + 1];
      }
  }
  // Expert and key of the largest value left; the same in every lane.
  __device__ __forceinline__ int next(int E, uint32_t &top) {
    top = wave_max_u32(key[0]);
    const unsigned long long holders = __ballot(key[0] == top);
    const int win = __builtin_ctzll(holders);  // (some lane holds the maximum)
    const int e = win * PER + __builtin_amdgcn_readlane(idx[0], win);
    const bool mine = lane_id() == win;
#pragma unroll
    for (int i = 0; i + 1 < PER; ++i) {
      key[i] = mine ? key[i + 1] : key[i];
      idx[i] = mine ? idx[i + 1] : idx[i];
    }
    key[PER - 1] = mine ? 0u : key[PER - 1];
    // k <= E, so an unpicked expert always exists; the clamp only guards against non-finite input
    return e < E ? e : 0;
  }
};

// The keys of a token's logits, lane l owning experts [l * PER, l * PER + PER).
template <int PER>
__device__ __forceinline__ void route_load_row(RowPicker<PER> &pick, const float *__restrict__ row, int E) {
  const int lane = lane_id();
  if (PER % 4 == 0 && (E & 3) == 0) {
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
      const int e0 = lane * PER + q * 4;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (e0 < E) v = *reinterpret_cast<const float4 *>(row + e0);  // E % 4 == 0: the four are inside together
      const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int u = 0; u < 4; ++u) pick.key[q * 4 + u] = e0 < E ? ordered_key(vv[u]) : 0u;
    }
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane * PER + i;
      pick.key[i] = e < E ? ordered_key(row[e]) : 0u;
    }
  }
}

// The k picks of one token whose logits' keys sit in `row`.  Lanes 0..k-1 write the picks (slot order = pick order) and
// their softmax weights renormalised over the picks.
template <int PER>
__device__ __forceinline__ void route_pick_registers(RowPicker<PER> &row, int E, int k, int t,
                                                     int32_t *__restrict__ topk_idx, float *__restrict__ topk_w,
                                                     int *also = nullptr) {  // also: a second place for the picks (LDS)
  const int lane = lane_id();
  row.sort();
  int my_e = 0;
  uint32_t my_key = 0, first = 0;
  for (int j = 0; j < k; ++j) {
    uint32_t top;
    const int e = row.next(E, top);
    if (j == 0) first = top;  // the largest logit: softmax shift
    if (lane == j) {
      my_e = e;
      my_key = top;
    }
  }
  const float x = expf(key_value(my_key) - key_value(first));
  float sum = 0.f;
  for (int j = 0; j < k; ++j) sum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j));  // slot order
  if (lane < k) {
    topk_idx[(size_t)t * k + lane] = my_e;
    if (also) also[t * k + lane] = my_e;
    topk_w[(size_t)t * k + lane] = x / sum;
  }
}

}  // namespace moe355
