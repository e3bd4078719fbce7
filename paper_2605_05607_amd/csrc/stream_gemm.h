// The forward pass of a small batch (decode): every expert has few rows, so the layer is a read of the busy experts'
// weights and nothing else.  Two kernels, no tile table, no work lists, no separate Combine.
//
// What bounds it: HBM (the weights of the busy experts), and below ~50 MB the latencies of the launches.  The tile
// kernels of gemm_bf16.h give one workgroup a 256-column panel over the whole reduction range; with a handful of busy
// experts that is a few dozen workgroups, each at the 50-60 GB/s one CU can pull.  Here a workgroup owns 32 h columns
// (GEMM-1) or 32 output columns (GEMM-2), its waves share the reduction range, and the weights go from memory straight
// into the registers the matrix instructions read: the packed tile stores an operand as one contiguous KiB, so there is
// nothing for the LDS to rearrange.  The waves' partial sums meet in the LDS, in wave order.
// Measured, whole step with route and tables, before (tile table + tile kernels + Combine) -> here: 0.7 GB of weights for
// one token 262 -> 126 us, 34 MB for 16 tokens 67.7 -> 28.8 us, 2.3 GB for 96 tokens 399 -> 335 us, 0.24 GB of FP8
// weights for 48 tokens 121 -> 85.6 us.
#pragma once
#include "gemm_bf16.h"
#include "route_pick.h"

namespace moe355 {

constexpr int kStreamTokens = 128;   // largest batch (GEMM-2 keeps one fp32 row of 32 columns per token and wave)
constexpr int kStreamExperts = 512;  // most local experts (GEMM-2 lists the busy ones in the LDS)
constexpr int kStreamWaves = 8;
constexpr int kStreamGroups = 8;  // most work groups per strip of GEMM-2

struct StreamArgs {
  const void *A;    // GEMM-1: x [T, K] (bf16, or codes); GEMM-2: h [rows, K]
  const void *Bp;   // packed tiles
  void *out;        // GEMM-1: h [rows, N]; GEMM-2: y [T, N] bf16
  float *partial;   // GEMM-2 with several groups: their sums, [group][strip][T][columns of the strip]
  int32_t *arrived; // groups that have stored theirs, per strip (cleared by GEMM-1: n_arrived of them, none for one group)
  int n_arrived;
  const int32_t *offsets, *perm;
  const float *topk_w;
  int32_t *error;   // status word of the workspace (cleared by GEMM-1: no wait can give up here)
  int T, k, e_lo, E_loc, P_cap;
  int K, N, n_ntiles, n_ktiles;
  const float *a_scale, *b_scale, *h_scale;  // FP8 only (see GemmArgs)
};

// Fragments of one k-step for up to NB 32-row blocks and NC 32-column blocks.
template <int NB, int NC>
struct StreamSlab {
  bf16x8 a[NB][4], b[NC][4];
};

template <bool FP8>
struct StreamElt {
  typedef typename std::conditional<FP8, uint8_t, bf16_t>::type type;
};

// Operands come in through buffer loads: the descriptor and everything that depends on the k-step are scalars, so a slab
// costs no vector registers for addresses (with flat addresses the compiler kept one per load and spilled).
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t stream_rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00027000);
}
__device__ __forceinline__ bf16x8 stream_fetch(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
__device__ __forceinline__ bf16x8 stream_fetch_once(rsrc_t r, uint32_t voff, uint32_t soff) {  // non-temporal
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 2));
}

// Loads of k-step kt.  b: the column block in tile 0 (lane * 16 is the lane's operand); a: the rows' matrix, a_off[mi]
// this lane's row plus khalf * 16, in bytes; row_bytes: bytes of a row.  A chunk past the row's end meets zeros in the
// packed tile and is read as zeros itself (an offset the descriptor's bound rejects), never from the next row.
template <bool FP8, bool WHOLE, int NB, int NC>
__device__ __forceinline__ void stream_load(StreamSlab<NB, NC> &s, rsrc_t a, const uint32_t (&a_off)[NB], rsrc_t b,
                                            uint32_t lane16, int kt, int row_bytes, int khalf16) {
#pragma unroll
  for (int j = 0; j < NC; ++j)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      s.b[j][kk] = stream_fetch_once(b, lane16 + kk * 1024, kt * kTileBytes + j * 4096);
#pragma unroll
  for (int mi = 0; mi < NB; ++mi)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const bool in = WHOLE || kt * 128 + kk * 32 + khalf16 < row_bytes;
      s.a[mi][kk] = stream_fetch(a, in ? a_off[mi] + kk * 32 : 0x80000000u, kt * 128);
    }
}

template <bool FP8, int NB, int NC>
__device__ __forceinline__ void stream_multiply(const StreamSlab<NB, NC> &s, f32x16 (&acc)[NB][NC]) {
  __builtin_amdgcn_sched_barrier(0);  // one slab after the other: its products, then its reload
#pragma unroll
  for (int mi = 0; mi < NB; ++mi)
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      if constexpr (FP8) {
        acc[mi][j] = mfma_fp8_pair(s.a[mi][0], s.a[mi][1], s.b[j][0], s.b[j][1], acc[mi][j]);
        acc[mi][j] = mfma_fp8_pair(s.a[mi][2], s.a[mi][3], s.b[j][2], s.b[j][3], acc[mi][j]);
      } else {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) acc[mi][j] = mfma_bf16(s.a[mi][kk], s.b[j][kk], acc[mi][j]);
      }
    }
  __builtin_amdgcn_sched_barrier(0);
}

template <int NB, int NC>
__device__ __forceinline__ void stream_clear(f32x16 (&acc)[NB][NC]) {
#pragma unroll
  for (int mi = 0; mi < NB; ++mi)
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][j][r] = 0.f;
}

// acc += k-steps [kt0, kt1) of one block, D slabs in flight.
template <bool FP8, int NB, int NC, int D>
__device__ __forceinline__ void stream_range(f32x16 (&acc)[NB][NC], rsrc_t a, const uint32_t (&a_off)[NB], rsrc_t b,
                                             uint32_t lane16, int kt0, int kt1, int row_bytes, int khalf16) {
  if (kt0 >= kt1) return;
  StreamSlab<NB, NC> s[D];
  if (kt1 * 128 > row_bytes) {  // the range ends with the row's last, partial k-step: that one on its own
    --kt1;
    stream_load<FP8, false>(s[0], a, a_off, b, lane16, kt1, row_bytes, khalf16);
    stream_multiply<FP8>(s[0], acc);
    if (kt0 == kt1) return;
  }
#pragma unroll
  for (int i = 0; i < D; ++i)
    if (i == 0 || kt0 + i < kt1) stream_load<FP8, true>(s[i], a, a_off, b, lane16, kt0 + i, row_bytes, khalf16);
  int kt = kt0;
  for (; kt + 2 * D <= kt1; kt += D) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      stream_multiply<FP8>(s[i], acc);
      stream_load<FP8, true>(s[i], a, a_off, b, lane16, kt + D + i, row_bytes, khalf16);
    }
  }
#pragma unroll
  for (int i = 0; i < D; ++i)
    if (kt + i < kt1) {
      stream_multiply<FP8>(s[i], acc);
      if (kt + D + i < kt1) stream_load<FP8, true>(s[i], a, a_off, b, lane16, kt + D + i, row_bytes, khalf16);
    }
#pragma unroll
  for (int i = 0; i < D - 1; ++i)
    if (kt + D + i < kt1) stream_multiply<FP8>(s[i], acc);
}

// The same for nb <= NB row blocks that hold rows: the usual single block runs the deeper pipeline D1 (its slabs are
// smaller; also, loads that are only sometimes issued would make every wait a wait for all of them).
template <bool FP8, int NB, int NC, int D1, int D2>
__device__ __forceinline__ void stream_blocks(f32x16 (&acc)[NB][NC], rsrc_t a, const uint32_t (&a_off)[NB], rsrc_t b,
                                              uint32_t lane16, int kt0, int kt1, int nb, int row_bytes, int khalf16) {
  if constexpr (NB == 2) {
    if (nb == 2) {
      stream_range<FP8, 2, NC, D2>(acc, a, a_off, b, lane16, kt0, kt1, row_bytes, khalf16);
      return;
    }
  }
  f32x16 one[1][NC];
  const uint32_t off[1] = {a_off[0]};
  stream_clear(one);
  stream_range<FP8, 1, NC, D1>(one, a, off, b, lane16, kt0, kt1, row_bytes, khalf16);
#pragma unroll
  for (int j = 0; j < NC; ++j) acc[0][j] = one[0][j];
}

// Token of a layout row (perm holds pair ids; clamped, so that a corrupt table stays inside x).
__device__ __forceinline__ int stream_pair(const StreamArgs &g, int row) {
  const int p = g.perm[row];
  return min(max(p, 0), g.T * g.k - 1);
}

// ------------------------------------------------------------------------------------------------
// GEMM-1: one workgroup per (32 h columns = one wave column of the packed tile, local expert).  Wave w of n takes the
// k-steps [w KT / n, (w + 1) KT / n); NB = 32-row blocks per pass (an expert with more rows takes
// another pass over its weights, which then come from the caches).
// ------------------------------------------------------------------------------------------------
template <bool FP8, int NB>
__global__ __launch_bounds__(kStreamWaves * 64, 2) void stream_gemm1_kernel(const StreamArgs g) {
  typedef typename StreamElt<FP8>::type elt_t;
  __shared__ float red[kStreamWaves][2][32][32];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, khalf = lane >> 5;
  const int c = blockIdx.x;
  if (c == 0 && blockIdx.y == 0) {
    if (tid == 0) *g.error = 0;
    for (int i = tid; i < g.n_arrived; i += kStreamWaves * 64) g.arrived[i] = 0;
  }
  const int base = g.offsets[g.e_lo];
  int le = blockIdx.y;
  if (NB > 1 && g.T > 32 * NB && g.E_loc <= 64) {
    // An expert may take several passes: the one with the most rows goes first.  (Where its number put it last, it was what the
    // launch waited for: 128 tokens with a skewed load on 32 of 256 experts of 7168 x 2048 180 -> 154 us, FP8 111 -> 97, 96 on
    // 16 of 128 of 4096 x 1536 104 -> 88; even loads within 1 %.  Up to 64 tokens, one pass each, looking for it costs an even
    // load 2.5 %, a skewed one gains 3 to 5 %: not done.)
    const int e = g.e_lo + min(lane, g.E_loc - 1), rows = max(g.offsets[e + 1] - g.offsets[e], 0);
    const int most = (int)(wave_max_u32((uint32_t)min(rows, 1 << 20) << 6 | (63 - lane)) & 63u);  // (of equals the first)
    const int first = 63 - most;
    le = le == 0 ? first : le - (le <= first);
  }
  const int start = min(max(g.offsets[g.e_lo + le] - base, 0), g.P_cap);
  const int rows_all = min(max(g.offsets[g.e_lo + le + 1] - base, 0), g.P_cap) - start;
  if (rows_all <= 0) return;  // whole workgroup
  const int kt0 = w * g.n_ktiles / kStreamWaves, kt1 = (w + 1) * g.n_ktiles / kStreamWaves;
  const rsrc_t b = stream_rsrc(static_cast<const unsigned char *>(g.Bp) +
                                   ((size_t)(le * g.n_ntiles + (c >> 2)) * g.n_ktiles) * kTileBytes + (c & 3) * 8192,
                               g.n_ktiles * kTileBytes - (c & 3) * 8192);
  const rsrc_t a = stream_rsrc(g.A, (uint32_t)g.T * g.K * sizeof(elt_t));
  for (int m0 = 0; m0 < rows_all; m0 += NB * 32) {
    const int rows = min(NB * 32, rows_all - m0);
    const int nb = (rows + 31) >> 5;
    uint32_t a_off[NB];
#pragma unroll
    for (int mi = 0; mi < NB; ++mi) {
      const int r = start + m0 + min(mi * 32 + l31, rows - 1);
      a_off[mi] = (uint32_t)(stream_pair(g, base + r) / g.k) * g.K * sizeof(elt_t) + khalf * 16;
    }
    f32x16 acc[NB][2];
    stream_clear(acc);
    stream_blocks<FP8, NB, 2, 3, 2>(acc, a, a_off, b, lane * 16, kt0, kt1, nb, g.K * (int)sizeof(elt_t), khalf * 16);
    // the waves' parts of one 32-row block at a time: rows that exist only
#pragma unroll
    for (int mi = 0; mi < NB; ++mi) {
      if (mi >= nb) break;  // (uniform)
      const int live = min(32, rows - mi * 32);
      if (mi > 0 || m0 > 0) __syncthreads();
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
        if (rl < live) {
          red[w][0][rl][l31] = acc[mi][0][r];
          red[w][1][rl][l31] = acc[mi][1][r];
        }
      }
      __syncthreads();
      for (int i = tid; i < live * 32; i += kStreamWaves * 64) {
        const int rl = i >> 5, cl = i & 31, col = c * 32 + cl;
        float gv = 0.f, uv = 0.f;
#pragma unroll
        for (int q = 0; q < kStreamWaves; ++q) {
          gv += red[q][0][rl][cl];
          uv += red[q][1][rl][cl];
        }
        if (col >= g.N) continue;
        const size_t row = (size_t)(start + m0 + mi * 32 + rl);
        if constexpr (FP8) {
          const float sx = g.a_scale[stream_pair(g, base + (int)row) / g.k];
          const float *bs = g.b_scale + (size_t)le * 2 * g.N;
          gv *= sx * bs[col];
          uv *= sx * bs[g.N + col];
          static_cast<uint8_t *>(g.out)[row * g.N + col] =
              to_e4m3((gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv))) * uv * __builtin_amdgcn_rcpf(g.h_scale[le]));
        } else {
          static_cast<bf16_t *>(g.out)[row * g.N + col] =
              (bf16_t)((gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv))) * uv);
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// GEMM-2 with Combine: one workgroup per strip of 32 output columns (and per group of the work, see below).  The k-steps
// of all busy experts of the strip form one list, cut into equal runs over the waves (and groups).  When a wave leaves an
// expert it adds weight * sum to its own fp32 row of each token in the LDS; at the end the waves' rows are added in wave order and written once: tokens without
// a local slot come out as zeros, and no row of o ever exists.  groups > 1 (strips too few to pull the weights at the
// chip's rate): every group stores its sums past the L2s (device-scope stores, as the resident kernels store h), counts itself
// for the strip, and the one that comes last adds them all in group order, every group's requested before the first is added
// (one after the other, the loads past the L2s took 0.8 us of six groups and one token, 2 us of eight groups and 128 tokens).
// A launch of its own for that sum took 4 to 5 us.
// ------------------------------------------------------------------------------------------------
// LDS: the waves' token rows | the busy list | token and weight of every local row
constexpr int stream_row_blocks(int T) { return T <= 32 ? 1 : 2; }  // NB: 32-row blocks per pass
// Entries of the busy list: a pass of 32 NB rows each, and every expert's last one may be partial.
constexpr int stream_passes(int P_cap, int E_loc, int nb) { return P_cap / (32 * nb) + E_loc; }
constexpr size_t stream2_lds_bytes(int T, int P_cap, int E_loc) {
  return (size_t)kStreamWaves * T * 32 * 4 + (size_t)stream_passes(P_cap, E_loc, stream_row_blocks(T)) * 16 +
         (size_t)P_cap * 8 + 16;
}

template <bool FP8, int NB>
__global__ __launch_bounds__(kStreamWaves * 64, 2) void stream_gemm2_kernel(const StreamArgs g) {
  typedef typename StreamElt<FP8>::type elt_t;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float *ysum = reinterpret_cast<float *>(smem);                                // [waves][T][32]
  int4 *seg = reinterpret_cast<int4 *>(ysum + kStreamWaves * g.T * 32);        // (expert, first row, rows, -)
  const int n_max = stream_passes(g.P_cap, g.E_loc, NB);                        // (more only in corrupt tables)
  int *row_tok = reinterpret_cast<int *>(seg + n_max);                          // [P_cap]
  float *row_w = reinterpret_cast<float *>(row_tok + g.P_cap);                  // [P_cap]
  int *n_seg_s = reinterpret_cast<int *>(row_w + g.P_cap);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, khalf = lane >> 5;
  const int c = blockIdx.x;
  const int base = g.offsets[g.e_lo];
  const int P = min(max(g.offsets[g.e_lo + g.E_loc] - base, 0), g.P_cap);
  float *mine = ysum + (size_t)w * g.T * 32;
  if (w == 0) {  // busy experts in order; one with more than 32 NB rows appears once per pass
    int n = 0;
    for (int e0 = 0; e0 < g.E_loc; e0 += 64) {
      const int le = e0 + lane;
      int start = 0, rows = 0;
      if (le < g.E_loc) {
        start = min(max(g.offsets[g.e_lo + le] - base, 0), P);
        rows = max(min(max(g.offsets[g.e_lo + le + 1] - base, 0), P) - start, 0);
      }
      const int passes = (rows + NB * 32 - 1) / (NB * 32);
      const int inc = wave_inclusive_scan(passes);
      for (int q = 0; q < passes && n + inc - passes + q < n_max; ++q)
        seg[n + inc - passes + q] = make_int4(le, start + q * NB * 32, min(NB * 32, rows - q * NB * 32), 0);
      n += __builtin_amdgcn_readlane(inc, 63);
    }
    if (lane == 0) *n_seg_s = min(n, n_max);
  }
  for (int r = tid; r < P; r += kStreamWaves * 64) {
    const int p = stream_pair(g, base + r);
    row_tok[r] = p / g.k;
    row_w[r] = g.topk_w[p];
  }
  for (int i = lane; i < g.T * 32; i += 64) mine[i] = 0.f;
  __syncthreads();
  const int KT = g.n_ktiles;
  const long long total = (long long)__builtin_amdgcn_readfirstlane(*n_seg_s) * KT;
  const int parts = kStreamWaves * gridDim.y, part = blockIdx.y * kStreamWaves + w;
  const int s0 = __builtin_amdgcn_readfirstlane((int)(total * part / parts));
  const int s1 = __builtin_amdgcn_readfirstlane((int)(total * (part + 1) / parts));

  const rsrc_t a = stream_rsrc(g.A, (uint32_t)P * g.K * sizeof(elt_t));
  for (int st = s0; st < s1;) {
    const int sg = st / KT, kt0 = st - sg * KT, kt1 = min(KT, kt0 + s1 - st);
    st += kt1 - kt0;
    const int4 v = seg[sg];
    const int le = __builtin_amdgcn_readfirstlane(v.x), start = __builtin_amdgcn_readfirstlane(v.y);
    const int rows = __builtin_amdgcn_readfirstlane(v.z), nb = (rows + 31) >> 5;
    uint32_t a_off[NB];
#pragma unroll
    for (int mi = 0; mi < NB; ++mi)
      a_off[mi] = (uint32_t)(start + min(mi * 32 + l31, rows - 1)) * g.K * sizeof(elt_t) + khalf * 16;
    const rsrc_t b = stream_rsrc(static_cast<const unsigned char *>(g.Bp) +
                                     ((size_t)(le * g.n_ntiles + (c >> 3)) * KT) * kTileBytes + (c & 7) * 4096,
                                 KT * kTileBytes - (c & 7) * 4096);
    float cs = 1.f;  // FP8: scale of the expert's h times the scale of this lane's column
    if constexpr (FP8) cs = g.h_scale[le] * g.b_scale[(size_t)le * g.N + min(c * 32 + l31, g.N - 1)];
    f32x16 acc[NB][1];
    stream_clear(acc);
    stream_blocks<FP8, NB, 1, 5, 3>(acc, a, a_off, b, lane * 16, kt0, kt1, nb, g.K * (int)sizeof(elt_t), khalf * 16);
    // weight * sum to this wave's token rows.  An expert's rows are in token order, and usually distinct tokens: all reads,
    // then all writes.  Picks that name an expert twice for a token put equal tokens side by side: one row after the other.
#pragma unroll
    for (int mi = 0; mi < NB; ++mi) {
      if (NB > 1 && mi >= nb) break;
      const int my = mi * 32 + l31;
      const int last = start + min(my, rows - 1);
      if (__any(l31 > 0 && my < rows && row_tok[last] == row_tok[last - (l31 > 0)])) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int kh = 0; kh < 2; ++kh) {
            const int rl = mi * 32 + (r >> 2) * 8 + kh * 4 + (r & 3);
            if (rl < rows && khalf == kh) {
              float *at = mine + row_tok[start + rl] * 32 + l31;
              *at = fmaf(FP8 ? acc[mi][0][r] * cs : acc[mi][0][r], row_w[start + rl], *at);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
          }
        continue;
      }
      int at[16];
      float sum[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = min(mi * 32 + (r >> 2) * 8 + khalf * 4 + (r & 3), rows - 1);
        at[r] = row_tok[start + rl] * 32 + l31;
        sum[r] = fmaf(FP8 ? acc[mi][0][r] * cs : acc[mi][0][r], row_w[start + rl], mine[at[r]]);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (mi * 32 + (r >> 2) * 8 + khalf * 4 + (r & 3) < rows) mine[at[r]] = sum[r];
    }
  }
  __syncthreads();
  const int tot = g.T * 8;  // four columns per thread
  const auto column_sum = [&](int i) {  // of this workgroup
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kStreamWaves; ++q) {
      const f32x4 o = *reinterpret_cast<const f32x4 *>(ysum + ((size_t)q * g.T + (i >> 3)) * 32 + (i & 7) * 4);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += o[u];
    }
    return v;
  };
  const auto store_y = [&](int i, const f32x4 &v) {
    const int col = c * 32 + (i & 7) * 4;
    if (col >= g.N) return;
    bf16x4 o;
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = (bf16_t)v[u];
    *reinterpret_cast<bf16x4 *>(static_cast<bf16_t *>(g.out) + (size_t)(i >> 3) * g.N + col) = o;
  };
  if (gridDim.y == 1 || total == 0) {  // (no local row: y is zero, nothing to hand over)
    if (blockIdx.y > 0) return;
    for (int i = tid; i < tot; i += kStreamWaves * 64) store_y(i, column_sum(i));
    return;
  }
  // two columns each; the last strip may have fewer than 32 columns, and no place is left for those it does not have
  uint64_t *partial = reinterpret_cast<uint64_t *>(g.partial);
  const int wide = min(32, g.N - c * 32);
  const auto place = [&](int group, int i) {
    return ((size_t)group * g.T * g.N + (size_t)c * 32 * g.T + (i >> 3) * wide + (i & 7) * 4) / 2;
  };
  for (int i = tid; i < tot; i += kStreamWaves * 64) {
    if ((i & 7) * 4 >= wide) continue;
    const f32x4 v = column_sum(i);
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    const u64x2 w = __builtin_bit_cast(u64x2, v);
    __hip_atomic_store(&partial[place(blockIdx.y, i)], w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&partial[place(blockIdx.y, i) + 1], w[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // acknowledged, every wave's, before the workgroup counts itself
  __syncthreads();
  if (tid == 0)
    *n_seg_s = __hip_atomic_fetch_add(&g.arrived[c], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.y - 1;
  __syncthreads();
  if (!*n_seg_s) return;  // whole workgroup
  for (int i = tid; i < tot; i += kStreamWaves * 64) {
    if ((i & 7) * 4 >= wide) continue;
    // every group's sum is requested before the first is added
    f32x4 sums[kStreamGroups];
#pragma unroll
    for (int q = 0; q < kStreamGroups; ++q) {
      if (q >= (int)gridDim.y) break;
      typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
      u64x2 w;
      w[0] = __hip_atomic_load(&partial[place(q, i)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      w[1] = __hip_atomic_load(&partial[place(q, i) + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sums[q] = __builtin_bit_cast(f32x4, w);
    }
    f32x4 v = sums[0];
#pragma unroll
    for (int q = 1; q < kStreamGroups; ++q) {
      if (q >= (int)gridDim.y) break;
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += sums[q][u];
    }
    store_y(i, v);
  }
}

}  // namespace moe355
