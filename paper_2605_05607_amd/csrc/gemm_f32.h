// Grouped fp32 GEMMs on the matrix cores (fp32 layers).
#pragma once
#include "stream_gemm.h"

namespace moe355 {

// ------------------------------------------------------------------------------------------------
// C[rows of one expert, 64 columns] = A * W_e in fp32 (v_mfma_f32_32x32x2_f32: fp32 products, fp32 sums).  GATED: 64 h
// columns from 64 gate and 64 up columns, h = silu(g) * u; else o = acc * row_w[row].  Weights are the unpacked "input x
// output" matrices.
//
// What bounds it: the fp32 matrix rate (1/16 of bf16's) on full experts, the weights or plain latency on small ones.  The
// instruction takes 64 cycles for 8 bytes per lane, so operands come straight from the caches without an LDS stage.
// A group is G reduction indices: lane l reads its row l % 32 at the G / 2 indices that start at G / 2 (l / 32) in 16-byte
// pieces and, of the weights, columns COLS (l % 32) .. + COLS at the same indices; instruction i then multiplies indices i and
// G / 2 + i.  The loads of a group are in flight while the group before it is multiplied (the counter of outstanding
// loads ends at 63: a second group in flight would not fit it).  The waves of the workgroup share the reduction range (the layers have few tiles: what fills the chip is
// cutting the sum) and meet in the LDS in wave order.
// Measured on 8 experts of 512 x 1024, GEMM-1 + GEMM-2 of 256 tokens: 76 + 95 us with 64 x 64 tiles on the vector ALU ->
// 29 + 17 us; step 192 -> 58 us, 8 tokens 189 -> 39 us, 2048 tokens 318 -> 195 us.
// ------------------------------------------------------------------------------------------------
template <int COLS>
__device__ __forceinline__ void f32_fetch(float (&v)[COLS], rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (COLS == 2) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    v[0] = __uint_as_float(t[0]);
    v[1] = __uint_as_float(t[1]);
  } else {
    v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  }
}

template <int MB, int NM, int G, int COLS>
struct F32Group {
  f32x4 a[MB][G / 8];
  float b[NM][G / 2][COLS];
};

// MB 32-row blocks and 32 COLS columns per workgroup.  An item of the work list covers 64 rows and 64 columns, so
// f32_parts workgroups share it, on the item's XCD.  NW waves.
constexpr int kF32Tiles = 1024;  // expected items from which on a workgroup takes a whole one
constexpr int f32_parts(int mb, int cols) { return (3 - mb) * (3 - cols); }
template <bool GATED, int MB, int COLS, int NW>
__global__ __launch_bounds__(NW * 64, 2) void gemm_f32_kernel(const GemmArgs g) {
  constexpr int NM = GATED ? 2 : 1, NJ = NM * COLS, G = MB == 2 ? 16 : 32, PARTS = f32_parts(MB, COLS);
  __shared__ float red[NW][NJ][32][32];
  const int part = (blockIdx.x >> 3) % PARTS, m_part = part % (3 - MB), n_part = part / (3 - MB);
  const int q = chunked_item((blockIdx.x & 7) | ((blockIdx.x >> 3) / PARTS) << 3, *g.n_items);
  if (q < 0) return;
  const int4 item = g.work[q];
  const int le = __builtin_amdgcn_readfirstlane(item.x);
  const int m0 = __builtin_amdgcn_readfirstlane(item.y) + m_part * 32;
  const int rows = (__builtin_amdgcn_readfirstlane(item.z) & kItemRowsMask) - m_part * 32;
  if (rows <= 0) return;  // whole workgroup
  const int n0 = (__builtin_amdgcn_readfirstlane(item.w) & ((1 << kTileShift) - 1)) * 64 + n_part * 32 * COLS;
  if (n0 >= g.N) return;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, khalf = lane >> 5;
  const int nb = min(MB, (rows + 31) >> 5);
  const int n_groups = (g.K + G - 1) / G;
  const int k0 = w * n_groups / NW, n_mine = (w + 1) * n_groups / NW - k0;  // this wave's groups
  // gate matrices of all local experts come first, then the up matrices (n_ktiles carries E_loc for this kernel)
  const size_t wsz = (size_t)g.K * g.N;
  const float *W0 = static_cast<const float *>(g.Bp) + (size_t)le * wsz + (size_t)k0 * G * g.N;
  const int k_len = max(0, min(n_mine * G, g.K - k0 * G));
  const uint32_t pitch = (uint32_t)g.N * 4;
  const uint32_t b_off = khalf * (G / 2) * pitch + min(n0 + COLS * l31, g.N - COLS) * 4;  // (columns past the end: not stored)
  const float *a_row[MB];
#pragma unroll
  for (int mi = 0; mi < MB; ++mi) {
    const int r = m0 + min(mi * 32 + l31, rows - 1);
    a_row[mi] = static_cast<const float *>(g.A) + (size_t)(g.row_map ? g.row_map[r] : r) * g.lda + k0 * G;
  }
  f32x16 acc[MB][NJ];
  stream_clear(acc);
  auto load = [&](F32Group<MB, NM, G, COLS> &s, int kg, auto whole) {
    // a descriptor per group: its offsets fit 32 bits whatever the size of the matrix
    const uint32_t bytes = (uint32_t)min(G, k_len - kg * G) * pitch;
    rsrc_t b[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) b[m] = stream_rsrc(W0 + m * g.n_ktiles * wsz + (size_t)kg * G * g.N, bytes);
#pragma unroll
    for (int i = 0; i < G / 2; ++i)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        if constexpr (decltype(whole)::value) {
          f32_fetch(s.b[m][i], b[m], b_off, (uint32_t)i * pitch);
        } else {  // indices past K: zeros, from offsets that the descriptor's bound rejects
          f32_fetch(s.b[m][i], b[m], b_off + (uint32_t)i * pitch, 0);
        }
      }
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
      for (int i = 0; i < G / 8; ++i) {
        const int kk = kg * G + khalf * (G / 2) + i * 4;
        s.a[mi][i] = *reinterpret_cast<const f32x4 *>(a_row[mi] + (decltype(whole)::value || kk < k_len ? kk : 0));
        if (!decltype(whole)::value && kk >= k_len) s.a[mi][i] = f32x4{0.f, 0.f, 0.f, 0.f};  // (an infinity times 0)
      }
  };
  auto multiply = [&](const F32Group<MB, NM, G, COLS> &s) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
      if (mi == 0 || nb > 1) {
#pragma unroll
        for (int i = 0; i < G / 2; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[mi][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                s.a[mi][i >> 2][i & 3], s.b[j / COLS][i][j % COLS], acc[mi][j], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int n_whole = k_len / G;
  F32Group<MB, NM, G, COLS> s0, s1;
  if (n_whole > 0) {
    const std::true_type whole;
    load(s0, 0, whole);
    for (int kg = 0; kg < n_whole; kg += 2) {  // (past the end: the last group again, not used)
      load(s1, min(kg + 1, n_whole - 1), whole);
      multiply(s0);
      load(s0, min(kg + 2, n_whole - 1), whole);
      if (kg + 1 < n_whole) multiply(s1);
    }
  }
  if (n_whole * G < k_len) {
    load(s0, n_whole, std::false_type());
    multiply(s0);
  }
#pragma unroll
  for (int mi = 0; mi < MB; ++mi) {
    if (mi >= nb) break;  // (uniform)
    if (mi > 0) __syncthreads();
    const int live = min(32, rows - mi * 32);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
      if (rl < live) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) red[w][j][rl][l31] = acc[mi][j][r];
      }
    }
    __syncthreads();
    for (int i = tid; i < live * 32; i += NW * 64) {
      const int rl = i >> 5, cl = i & 31;
      float v[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        v[j] = 0.f;
#pragma unroll
        for (int p = 0; p < NW; ++p) v[j] += red[p][j][rl][cl];
      }
      const size_t grow = (size_t)(m0 + mi * 32 + rl);
      const int col = n0 + COLS * cl;
      if (col >= g.N) continue;
      float *out = static_cast<float *>(g.out) + grow * g.ldo + col;
      const float wgt = GATED ? 1.f : g.row_w[grow];
#pragma unroll
      for (int c = 0; c < COLS; ++c)
        out[c] = GATED ? (v[c] / (1.0f + expf(-v[c]))) * v[NJ - COLS + c] : v[c] * wgt;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// The same products where the batch is small: no tile table (an expert's rows come from the dispatch tables), one workgroup of
// eight waves per (32 columns, unit), each wave with an eighth of the reduction range.  A unit is an expert with up to 32 MB rows,
// or 32 rows of one with more; the workgroups of a strip take turns over the units of the whole load, which they number from
// `offsets`.  (With workgroups that each keep to one expert, a large one was turn after turn of a few of them, and the
// experts without rows scattered the others over the CUs.  Forward call, 414 tokens on 8 of 64 experts of 1024 x 1024, 200 rows
// on one of them, 82 -> 49 us, 430 on 16 of 128 of 512 x 1024, 400 rows on one, 127 -> 52; tile kernels 71 and 73.)
// What bounds it is the latency of the weight stream, so a wave has D groups of 16 reduction indices in flight: with D = 4 all of a
// range of 512 at once.  MB = 3: experts of 32 to 96 rows in one pass over their weights; such experts are hardly ever empty, so
// the first weights of each are requested before the tables have been read.
// Measured, step with weights from HBM, against the kernels above with their tile table: 8 tokens on 8 experts of 512 x 1024
// 41.1 -> 30.1 us, 32 on 8 of 2048 x 2048 178 -> 106 (402 MB of weights), 64 on 16 of 264 x 2000 88 -> 51; MB = 3: 256 tokens on 8
// experts of 512 x 1024 59.9 -> 54.2 us.
// ------------------------------------------------------------------------------------------------
struct F32Args {
  const float *A, *W;  // GEMM-1: x [T, K] and the gate, then the up matrices; GEMM-2: h [rows, K] and the down matrices
  float *out;          // h [rows, N]; weighted rows o [rows, N]
  const int32_t *offsets, *perm;
  const float *topk_w;
  int32_t *error;      // status word of the workspace (cleared by GEMM-1: no wait can give up here)
  int T, k, e_lo, E_loc, P_cap, K, N;
  int most;            // units of any load
};

// Sum of the lanes up to and including this one, by data-parallel moves: within the rows of 16 lanes, then the rows' totals.
// (Every unit starts with it: with lane permutes through the LDS port the two launches of a layer of 8 to 256 columns took 1 us more.)
__device__ __forceinline__ int f32_lane_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Unit `u` of the load: its expert, that expert's first row and rows, the unit's number in the expert; more: whether there may
// be a unit u + step.  An expert with up to 32 MB rows is one unit, one with more has a unit per 32 rows.  MB > 1 (up to 64
// experts): units 0 .. E_loc - 1 are the first of each expert, also of one without rows, the others follow.
struct F32Unit { int le, start, rows, number; bool more; };
template <int MB>
__device__ __forceinline__ F32Unit f32_unit(const F32Args &g, int u, int step, int base, int lane) {
  F32Unit r{-1, 0, 0, 0, false};
  const bool some_left = u + step < g.most;
  const auto bounds = [&](int e0) {
    const int32_t *at = g.offsets + g.e_lo + min(e0 + lane, g.E_loc - 1);
    return int2{at[0], at[1]};
  };
  int2 next = bounds(0);
  for (int e0 = 0; e0 < g.E_loc; e0 += 64) {
    const int2 cur = next;
    if (e0 + 64 < g.E_loc) next = bounds(e0 + 64);
    const int start = min(max(cur.x - base, 0), g.P_cap);
    const int rows = e0 + lane < g.E_loc ? max(min(max(cur.y - base, 0), g.P_cap) - start, 0) : 0;
    const int n = MB > 1 ? (rows > 32 * MB ? (rows - 1) >> 5 : 0) : (rows + 31) >> 5;
    const int upto = f32_lane_scan(n), all = __builtin_amdgcn_readlane(upto, 63);
    int at = u;  // MB > 1: the lane of the expert whose first unit it is
    if (MB == 1 || u >= g.E_loc) {
      const int i = MB > 1 ? u - g.E_loc : u;
      if (i >= all) {
        u -= all;
        continue;
      }
      at = __builtin_ctzll(__ballot(upto > i));
      r.number = i - __builtin_amdgcn_readlane(upto - n, at) + (MB > 1 ? 1 : 0);
    }
    r.le = e0 + at;
    r.start = __builtin_amdgcn_readlane(start, at);
    r.rows = __builtin_amdgcn_readlane(rows, at);
    r.more = some_left && (u + step < all + (MB > 1 ? g.E_loc : 0) || e0 + 64 < g.E_loc);
    break;
  }
  return r;
}

constexpr int kF32Waves = 8;
// OCC: waves per SIMD that the registers are cut for.
template <bool GATED, int MB, int D, int OCC>
__global__ __launch_bounds__(kF32Waves * 64, OCC) void gemm_f32_direct_kernel(const F32Args g) {
  constexpr int NM = GATED ? 2 : 1, G = 16, NW = kF32Waves;
  __shared__ float red[NW][NM][32][32];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n0 = blockIdx.x * 32;
  if (GATED && threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0) *g.error = 0;
  const int n_groups = (g.K + G - 1) / G;
  const int k0 = w * n_groups / NW, n_mine = (w + 1) * n_groups / NW - k0;  // this wave's groups
  const size_t wsz = (size_t)g.K * g.N;
  const float *W0 = g.W + (size_t)min((int)blockIdx.y, g.E_loc - 1) * wsz + (size_t)k0 * G * g.N;
  const int k_len = max(0, min(n_mine * G, g.K - k0 * G)), n_whole = k_len / G;
  const uint32_t pitch = (uint32_t)g.N * 4;
  int l31 = threadIdx.x & 31, khalf = (threadIdx.x >> 5) & 1;
  uint32_t b_off = khalf * (G / 2) * pitch + min(n0 + l31, g.N - 1) * 4;  // (columns past the end: not stored)
  const float *a_row[MB];
  F32Group<MB, NM, G, 1> s[D];
  const std::true_type whole;
  auto load_b = [&](F32Group<MB, NM, G, 1> &s, int kg, auto whole) {
    // a descriptor per group: its offsets fit 32 bits whatever the size of the matrix
    const uint32_t bytes = (uint32_t)min(G, k_len - kg * G) * pitch;
    rsrc_t b[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) b[m] = stream_rsrc(W0 + m * g.E_loc * wsz + (size_t)kg * G * g.N, bytes);
#pragma unroll
    for (int i = 0; i < G / 2; ++i)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        if constexpr (decltype(whole)::value) {
          f32_fetch(s.b[m][i], b[m], b_off, (uint32_t)i * pitch);
        } else {  // indices past K: zeros, from offsets that the descriptor's bound rejects
          f32_fetch(s.b[m][i], b[m], b_off + (uint32_t)i * pitch, 0);
        }
      }
  };
  auto load_a = [&](F32Group<MB, NM, G, 1> &s, int kg, auto whole) {
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
      for (int i = 0; i < G / 8; ++i) {
        const int kk = kg * G + khalf * (G / 2) + i * 4;
        s.a[mi][i] = *reinterpret_cast<const f32x4 *>(a_row[mi] + (decltype(whole)::value || kk < k_len ? kk : 0));
        if (!decltype(whole)::value && kk >= k_len) s.a[mi][i] = f32x4{0.f, 0.f, 0.f, 0.f};  // (an infinity times 0)
      }
  };
  bool early = MB > 1 && (int)blockIdx.y < g.E_loc;  // the first weights ahead of the tables
  if (early) {
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (i < n_whole) load_b(s[i], i, whole);
  }
  const int base = g.offsets[g.e_lo];
  bool more = true, used = false;  // used: the LDS, by an earlier unit
  for (int u = blockIdx.y; more; u += gridDim.y) {
    const F32Unit e = f32_unit<MB>(g, u, gridDim.y, base, fresh_lane());
    more = e.more;
    if (e.rows <= 0) {  // (uniform)
      early = false;
      continue;
    }
    W0 = g.W + (size_t)e.le * wsz + (size_t)k0 * G * g.N;
    const int tid = w * 64 + fresh_lane();  // (what hangs on the lane is not kept across the units: registers)
    l31 = tid & 31;
    khalf = (tid >> 5) & 1;
    b_off = khalf * (G / 2) * pitch + min(n0 + l31, g.N - 1) * 4;
    const int start = e.start, m0 = e.number * 32;
    const int rows = e.rows <= 32 * MB ? e.rows : min(32, e.rows - m0), nb = (rows + 31) >> 5;
#pragma unroll
    for (int mi = 0; mi < MB; ++mi) {
      const int r = start + m0 + min(mi * 32 + l31, rows - 1);
      a_row[mi] = g.A + (size_t)(GATED ? min(max(g.perm[base + r], 0), g.T * g.k - 1) / g.k : r) * g.K + k0 * G;
    }
    f32x16 acc[MB][NM];
    stream_clear(acc);
    auto load = [&](F32Group<MB, NM, G, 1> &s, int kg, auto whole) {
      load_b(s, kg, whole);
      load_a(s, kg, whole);
    };
    auto multiply = [&](const F32Group<MB, NM, G, 1> &s) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mi = 0; mi < MB; ++mi)
        if (mi < nb) {
#pragma unroll
          for (int i = 0; i < G / 2; ++i)
#pragma unroll
            for (int m = 0; m < NM; ++m)
              acc[mi][m] = __builtin_amdgcn_mfma_f32_32x32x2f32(s.a[mi][i >> 2][i & 3], s.b[m][i][0], acc[mi][m], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (i < n_whole) {
        if (!early) load_b(s[i], i, whole);
        load_a(s[i], i, whole);
      }
    early = false;
    int kg = 0;
    for (; kg + 2 * D <= n_whole; kg += D) {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        multiply(s[i]);
        load(s[i], kg + D + i, whole);
      }
    }
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (kg + i < n_whole) {
        multiply(s[i]);
        if (kg + D + i < n_whole) load(s[i], kg + D + i, whole);
      }
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
      if (kg + D + i < n_whole) multiply(s[i]);
    if (n_whole * G < k_len) {
      load(s[0], n_whole, std::false_type());
      multiply(s[0]);
    }
    // the waves' parts of one 32-row block at a time, in wave order
#pragma unroll
    for (int mi = 0; mi < MB; ++mi) {
      if (mi >= nb) break;  // (uniform)
      const int live = min(32, rows - mi * 32);
      if (mi > 0 || used) __syncthreads();  // (the block before is done with the LDS)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
        if (rl < live) {
#pragma unroll
          for (int m = 0; m < NM; ++m) red[w][m][rl][l31] = acc[mi][m][r];
        }
      }
      __syncthreads();
      for (int i = tid; i < live * 32; i += NW * 64) {
        const int rl = i >> 5, cl = i & 31;
        float v[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          v[m] = 0.f;
#pragma unroll
          for (int p = 0; p < NW; ++p) v[m] += red[p][m][rl][cl];
        }
        const int row = start + m0 + mi * 32 + rl, col = n0 + cl;
        if (col >= g.N) continue;
        g.out[(size_t)row * g.N + col] = GATED ? (v[0] / (1.0f + expf(-v[0]))) * v[NM - 1]
                                               : v[0] * g.topk_w[min(max(g.perm[base + row], 0), g.T * g.k - 1)];
      }
    }
    used = true;
  }
}

}  // namespace moe355
