// moe_fused_forward and its building blocks: weight packing, tile table, grouped SwiGLU GEMMs (GEMM-1 and
// GEMM-2 of Sec. II-A) with the token gather fused into GEMM-1's operand load (Dispatch of Sec. II-A without a
// materialised copy), the gate weight applied in GEMM-2's epilogue (Sec. III-C), and the per-token reduction
// with a single write-back (Combine; the one-GPU form of the in-switch reduction of Sec. II-C).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>

#include "backward_kernels.h"
#include "combine_kernels.h"
#include "fp8_kernels.h"
#include "gemm_bf16.h"
#include "gemm_f32.h"
#include "pack_kernels.h"
#include "prep_kernel.h"
#include "stream_gemm.h"
#include "wgrad_bf16.h"

namespace moe355 {

// ------------------------------------------------------------------------------------------------
// Host-side launch helpers
// ------------------------------------------------------------------------------------------------
struct Ws {
  int32_t *header, *tickets, *row_tok, *row_sole, *tile_ready, *row_tile, *tile_done, *arrived;
  int4 *work1, *work2;
  float *row_w;
  void *h;
  float *o;
};

static Ws carve(void *workspace, const FwdLayout &L) {
  unsigned char *b = static_cast<unsigned char *>(workspace);
  Ws w;
  w.header = reinterpret_cast<int32_t *>(b + L.header);
  w.tickets = reinterpret_cast<int32_t *>(b + L.tickets);
  w.work1 = reinterpret_cast<int4 *>(b + L.work1);
  w.work2 = reinterpret_cast<int4 *>(b + L.work2);
  w.row_tok = reinterpret_cast<int32_t *>(b + L.row_tok);
  w.row_w = reinterpret_cast<float *>(b + L.row_w);
  w.row_sole = reinterpret_cast<int32_t *>(b + L.row_sole);
  w.tile_ready = reinterpret_cast<int32_t *>(b + L.tile_ready);
  w.row_tile = reinterpret_cast<int32_t *>(b + L.row_tile);
  w.tile_done = reinterpret_cast<int32_t *>(b + L.tile_done);
  w.arrived = reinterpret_cast<int32_t *>(b + L.arrived);
  w.h = b + L.h;
  w.o = reinterpret_cast<float *>(b + L.o);
  return w;
}

// LDS of the tile-table kernel: four (with the row -> tile map: five) per-expert arrays, a counter and the scan scratch.
static size_t prep_lds_bytes(const Derived &dv, bool combine_tables) {
  return (size_t)((combine_tables ? 5 : 4) * dv.E_loc + 2 + 1 + 17) * sizeof(int);
}

// Whether the tile-table kernel also makes the FP8 codes: not where its tables take so much LDS that few workgroups fit a CU.
constexpr size_t kTokenCodesLds = 16 * 1024;
static bool codes_with_table(const moe_shape *s, const Derived &dv) {
  return s->T <= 1 << 22 && prep_lds_bytes(dv, false) <= kTokenCodesLds;
}

// sole != nullptr: also mark the rows GEMM-2 may write straight to y (see the GEMM-2 epilogue);
// combine_tables: also the row -> M tile map and the cleared GEMM-2 counters of the resident kernel's Combine stage;
// tokens.codes != nullptr: also the FP8 codes of the tokens that have a local slot
static int launch_prep(const moe_shape *s, const Derived &dv, const moe_dispatch *tb, const int32_t *topk_idx,
                       const float *topk_w, const Ws &w, int32_t *sole, hipStream_t st, bool combine_tables = false,
                       const TokenCodes &tokens = TokenCodes{}) {
  static_assert((5 * kMaxExperts + 20) * sizeof(int) <= 96 * 1024, "per-expert tables fit the LDS");
  const int blocks = (int)std::min<int64_t>(512, std::max<int64_t>(1, (dv.P_cap + 255) / 256));
  const int token_blocks = tokens.codes ? s->T : 0;
  const auto launch = [&](auto kernel, std::atomic<uint64_t> &done) {
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(kernel), 96 * 1024, done)) return (int)MOE_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3(2 * blocks + token_blocks), dim3(256), prep_lds_bytes(dv, combine_tables), st,
                       tb->offsets, tb->perm, topk_w, s->T, s->k, dv.e_lo, dv.E_loc, dv.bm, (int)dv.P_cap, dv.max_mtiles,
                       dv.nt1, dv.nt2, blocks, w.header, w.tickets, w.work1, w.work2, w.row_tok, w.row_w, topk_idx, sole,
                       w.tile_ready, combine_tables ? w.row_tile : nullptr, combine_tables ? w.tile_done : nullptr, tokens);
    return launch_status();
  };
  static std::atomic<uint64_t> done{0}, done_q{0};
  return tokens.codes ? launch(&fwd_prep_kernel<true>, done_q) : launch(&fwd_prep_kernel<false>, done);
}

// Compute units of the current device, looked up once per device (0 on failure).
static int compute_units() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) return 0;
  cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

// FP8 form of the GEMMs: quantised x with its per-token scales, the column scales that follow the packed tiles,
// and the per-expert scale of h.
struct Fp8Operands {
  const uint8_t *xq;
  const float *x_scale, *gu_scale, *down_scale, *h_scale;
};

static size_t fp8_tile_bytes(const moe_shape *s, const Derived &dv, int which) {
  if (which == 0) return (size_t)dv.E_loc * ceil_div(s->f, kBN / 2) * ceil_div(s->d, kFp8KStep) * kTileBytes;
  return (size_t)dv.E_loc * ceil_div(s->d, kBN) * ceil_div(s->f, kFp8KStep) * kTileBytes;
}

// The per-item GEMM kernel: one workgroup per item of the list, `far` (A has 4 GiB or more) with 64-bit row addresses.
template <bool GATED, bool FP8, bool TRAIN, bool FAR, bool BESIDE>
static bool launch_items_(const GemmArgs &g, dim3 grid, hipStream_t st) {
  static std::atomic<uint64_t> done{0};
  const auto kernel = &gemm_bf16_kernel<GATED, FP8, TRAIN, FAR, BESIDE>;
  const int lds = BESIDE ? kGemmLdsBeside : kGemmLds;  // more than the default dynamic limit: raised per function
  if (!allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds, done)) return false;
  hipLaunchKernelGGL(kernel, grid, dim3(kGemmThreads), lds, st, g);
  return true;
}
template <bool GATED, bool FP8, bool TRAIN, bool BESIDE = false>
static int launch_items(const GemmArgs &g, bool far, dim3 grid, hipStream_t st) {
  const bool ok = !FP8 && far ? launch_items_<GATED, FP8, TRAIN, !FP8, BESIDE>(g, grid, st)
                              : launch_items_<GATED, FP8, TRAIN, false, BESIDE>(g, grid, st);
  return ok ? launch_status() : (int)MOE_ERR_HIP;
}

// A resident kernel: one workgroup per CU (each takes most of a CU's LDS).
template <void (*KERNEL)(PipelineArgs)>
static int launch_resident(const PipelineArgs &pa, hipStream_t st) {
  static std::atomic<uint64_t> done{0};
  const int n_cu = compute_units();
  if (n_cu < 1 || !allow_dynamic_lds(reinterpret_cast<const void *>(KERNEL), kGemmLds, done)) return MOE_ERR_HIP;
  hipLaunchKernelGGL(KERNEL, dim3((unsigned)n_cu), dim3(kGemmThreads), kGemmLds, st, pa);
  return launch_status();
}

// GEMM-1 (gated) then GEMM-2 on the rows described by the tile table.  a1 / a1_map select the A operand of
// GEMM-1: the token matrix with the row -> token map (fused gather) or a materialised copy (map == nullptr).
static int launch_gemms(const moe_shape *s, const Derived &dv, const void *a1, const int32_t *a1_map, int a1_ld,
                        const void *packed_gu, const void *packed_down, const Ws &w, const int32_t *sole, void *y,
                        hipStream_t st, void *const *events = nullptr, bool pipelined = false,
                        const Fp8Operands *q = nullptr, void *keep_gu = nullptr, float *keep_o = nullptr,
                        int max_polls = kMaxPolls, int wait_extra = 0, const moe_dispatch *combine_tb = nullptr,
                        const int32_t *topk_idx = nullptr) {
  auto mark = [&](int i) {
    if (events && events[i]) (void)hipEventRecord((hipEvent_t)events[i], st);
  };
  GemmArgs g1{};
  g1.A = a1; g1.row_map = a1_map; g1.Bp = packed_gu; g1.out = w.h; g1.row_w = nullptr;
  g1.row_sole = nullptr; g1.y = nullptr;
  g1.n_items = w.header + 0; g1.work = w.work1;
  int ldh = h_pitch(s, q ? 1 : dv.elt);
  if (q && dv.P_cap * ldh >= (int64_t)1 << 32) {  // (padding the rows would take them out of reach of 32-bit offsets)
    ldh = s->f;
    pipelined = false;
  }
  g1.K = s->d; g1.N = s->f; g1.lda = a1_ld; g1.ldo = ldh;
  GemmArgs g2 = g1;
  g2.A = w.h; g2.row_map = nullptr; g2.Bp = packed_down; g2.out = w.o; g2.row_w = w.row_w;
  g2.row_sole = sole; g2.y = y;
  g2.K = s->f; g2.N = s->d; g2.lda = ldh; g2.ldo = s->d;
  g2.n_items = w.header + 3; g2.work = w.work2;
  // (bf16 only: an operand has less than 2^32 elements, see forward_common)
  const bool far1 = (a1_map ? (int64_t)s->T : dv.P_cap) * a1_ld * 2 >= (int64_t)1 << 32;
  const bool far2 = dv.P_cap * ldh * 2 >= (int64_t)1 << 32;
  if (keep_gu) {  // training forward: g and u are kept, and every weighted row goes to the kept o
    g1.aux = keep_gu;
    g2.out = keep_o;
    g2.keep_rows = 1;
  }
  const auto grid_of = [&](int nt) { return dim3((unsigned)(((size_t)dv.max_mtiles * nt + 255) / 256 * 256)); };
  if (s->dtype == MOE_BF16) {
    const int step = q ? kFp8KStep : kBK;
    if (q) {
      g1.A = q->xq; g1.a_scale = q->x_scale; g1.b_scale = q->gu_scale; g1.h_scale = q->h_scale;
      g2.b_scale = q->down_scale; g2.h_scale = q->h_scale;
    }
    g1.n_ntiles = ceil_div(s->f, kBN / 2); g1.n_ktiles = ceil_div(s->d, step);
    g2.n_ntiles = ceil_div(s->d, kBN);     g2.n_ktiles = ceil_div(s->f, step);
    int rc;
    if (pipelined) {
      PipelineArgs pa{};
      pa.g1 = g1; pa.g2 = g2;
      pa.tickets = w.tickets; pa.tile_ready = w.tile_ready; pa.error = w.header + 24; pa.nt1 = dv.nt1 + wait_extra;
      pa.max_polls = max_polls;
      const bool far = far1 || far2;
#define MOE355_RESIDENT(KERNEL_) (far ? launch_resident<KERNEL_<true>>(pa, st) : launch_resident<KERNEL_<false>>(pa, st))
      if (q) {
        rc = launch_resident<gemm_fp8_pipeline_kernel>(pa, st);
      } else if (keep_gu) {
        rc = MOE355_RESIDENT(gemm_train_pipeline_kernel);
      } else if (combine_tb) {
        // Combine as the third stage of the same launch (wait_extra also raises its target, for the give-up test)
        pa.tile_done = w.tile_done; pa.row_tile = w.row_tile;
        pa.topk_idx = topk_idx; pa.inv_perm = combine_tb->inv_perm; pa.offsets = combine_tb->offsets;
        pa.header = w.header;
        pa.T = s->T; pa.k = s->k; pa.e_lo = dv.e_lo; pa.E_loc = dv.E_loc; pa.P_cap = (int)dv.P_cap;
        pa.nt2 = dv.nt2 + wait_extra; pa.n_mtiles_cap = dv.max_mtiles;
        rc = MOE355_RESIDENT(gemm_bf16_combine_kernel);
      } else {
        rc = MOE355_RESIDENT(gemm_bf16_pipeline_kernel);
      }
#undef MOE355_RESIDENT
      mark(2);
      mark(3);
      return rc;
    }
    if (q) rc = launch_items<true, true, false>(g1, false, grid_of(dv.nt1), st);
    else if (keep_gu) rc = launch_items<true, false, true>(g1, far1, grid_of(dv.nt1), st);
    else rc = launch_items<true, false, false>(g1, far1, grid_of(dv.nt1), st);
    mark(2);
    if (rc != MOE_OK) return rc;
    if (q) rc = launch_items<false, true, false>(g2, false, grid_of(dv.nt2), st);
    else rc = launch_items<false, false, false>(g2, far2, grid_of(dv.nt2), st);
    mark(3);
    return rc;
  }
  g1.n_ntiles = ceil_div(s->f, kFBN); g1.n_ktiles = dv.E_loc;
  g2.n_ntiles = ceil_div(s->d, kFBN); g2.n_ktiles = dv.E_loc;
  // Tile by the expected number of 64 x 64 items (mean load): whole items where there are four per CU, else quarters, so
  // that no CU has two workgroups while others have one (each is ~10 us of matrix-core time); GEMM-2, which has fewer,
  // eight waves per workgroup below one item per CU.
  const double rows = (double)s->T * s->k * dv.E_loc / s->E;
  const double mtiles = std::min<double>(dv.E_loc, rows) + rows / kFBM;
  const auto launch = [&](auto kernel, int nt, int parts, int waves, const GemmArgs &g) {
    dim3 grid = grid_of(nt);
    grid.x *= parts;
    hipLaunchKernelGGL(kernel, grid, dim3(waves * 64), 0, st, g);
  };
  if (mtiles * dv.nt1 >= kF32Tiles) launch(gemm_f32_kernel<true, 2, 2, 4>, dv.nt1, f32_parts(2, 2), 4, g1);
  else launch(gemm_f32_kernel<true, 1, 1, 4>, dv.nt1, f32_parts(1, 1), 4, g1);
  int rc = launch_status();
  mark(2);
  if (rc != MOE_OK) return rc;
  if (mtiles * dv.nt2 >= kF32Tiles) launch(gemm_f32_kernel<false, 2, 2, 4>, dv.nt2, f32_parts(2, 2), 4, g2);
  else if (mtiles * dv.nt2 >= kF32Tiles / 4) launch(gemm_f32_kernel<false, 1, 2, 4>, dv.nt2, f32_parts(1, 2), 4, g2);
  else launch(gemm_f32_kernel<false, 1, 1, 8>, dv.nt2, f32_parts(1, 1), 8, g2);
  mark(3);
  return launch_status();
}

// fp32 layers of small batches: the kernels without a tile table (gemm_f32_direct_kernel); 32-row blocks per workgroup of
// GEMM-1, 0 = the tile kernels.  A load cannot be seen here, so each line holds for even loads and for the skewed ones of the
// workload generator (power law, the hottest rank local).  Time of this form's forward call over the tile kernels', median (and
// the tenth of the layers above), 5200 random layers of 256 to 2048 columns and 1 to 128 local experts, weights from HBM:
//                                                                    even          skewed
//   up to 24 rows per expert, 1 to 32 tokens, up to 3072 strips       0.78 (0.89)   0.80 (0.90)   (3500 strips: up to 1.27)
//     33 to 256 tokens, up to 1536 strips of 32 columns               0.72 (0.89)   0.82 (0.92)
//     257 to 768                                                      0.68 (0.81)   0.82 (0.95)
//     769 to 1536 (beyond: up to 1.25 under skew)                     0.67 (0.76)   0.88 (0.99)
//     more strips (tile kernels), 33 to 512 tokens: the weights come
//     from enough workgroups in either form, latency counts less      0.84 (1.15)   0.89 (1.12)
//   more than 24 rows, up to 384 tokens, few workgroups: one block    0.88 (0.96)   0.87 (0.96)
//   three blocks, an even load is one unit of up to 96 rows per
//   expert in nearly full rounds of one workgroup per CU: one round
//   of experts with up to 40 rows                                     0.89 (0.99)   0.84 (1.01)
//     with 62 to 87, i.e. two 64-row tiles for many                   0.78 (0.95)   0.94 (1.01)
//     with 40 to 62, which a tile holds (tile kernels)                1.01 (1.05)   0.94 (1.05)
//   more rounds, up to 36 rows                                        0.86 (0.96)   0.86 (0.93)
//     more rows (tile kernels): 1.00 to 1.11 even, 1.05 to 1.17 skewed
// Three blocks not with columns of 376 to 424 in GEMM-2 either, which are all prologue and sum (1.10 to 1.23).  One block: 24 to 32
// rows on 16 of 936 x 440, where many experts have more than 32, 1.09.
int f32_direct_blocks(const moe_shape *s, const Derived &dv) {
  if (s->dtype != MOE_F32) return 0;
  const int64_t strips = (int64_t)dv.E_loc * ceil_div(s->f, 32), widest = (int64_t)dv.E_loc * ceil_div(std::max(s->d, s->f), 32);
  const double rows = (double)s->T * s->k / s->E;
  if (rows <= 24.0) return s->T <= 1536 && widest <= (s->T <= 32 ? 3072 : 1536) ? 1 : 0;
  if (s->T > 384) return 0;
  if (strips * std::ceil(rows / 32) < 256 && strips * std::ceil(1.25 * rows / 32) < 384) return 1;
  const bool full_rounds = strips >= 192 && strips <= 1024 && (strips <= 256 || strips >= 0.9 * 256 * std::ceil(strips / 256.0));
  const bool one_tile = rows > 40 && rows < 62, pays = strips > 256 ? rows <= 36 : rows <= 87 && !one_tile;
  return s->d >= 512 && s->f >= 512 && pays && full_rounds ? 3 : 0;
}

static int launch_f32_direct(const moe_shape *s, const Derived &dv, int blocks, const void *x, const float *topk_w,
                             const moe_dispatch *tb, const void *packed_gu, const void *packed_down, const Ws &w,
                             hipStream_t st, void *const *events) {
  auto mark = [&](int i) {
    if (events && events[i]) (void)hipEventRecord((hipEvent_t)events[i], st);
  };
  F32Args g1{};
  g1.A = static_cast<const float *>(x); g1.W = static_cast<const float *>(packed_gu); g1.out = static_cast<float *>(w.h);
  g1.offsets = tb->offsets; g1.perm = tb->perm; g1.topk_w = topk_w; g1.error = w.header + 24;
  g1.T = s->T; g1.k = s->k; g1.e_lo = dv.e_lo; g1.E_loc = dv.E_loc; g1.P_cap = (int)dv.P_cap;
  g1.K = s->d; g1.N = s->f;
  F32Args g2 = g1;
  g2.A = static_cast<const float *>(w.h); g2.W = static_cast<const float *>(packed_down); g2.out = w.o;
  g2.K = s->f; g2.N = s->d;
  const double local = (double)s->T * s->k * dv.E_loc / s->E;  // rows of an even load
  const auto launch = [&](auto kernel, int mb, int resident, F32Args g) {
    // units of any load, or those of an even one and a quarter more, or what the chip holds at once; workgroups take turns
    const int strips = ceil_div(g.N, 32);
    const int64_t most = (mb > 1 ? dv.E_loc : std::min<int64_t>(dv.E_loc, dv.P_cap)) + dv.P_cap / 32;
    g.most = (int)most;
    const int64_t even = mb > 1 ? dv.E_loc : (int64_t)std::ceil(1.25 * (std::min<double>(dv.E_loc, local) + local / 32));
    const int64_t units = std::min(most, std::max<int64_t>(even, ceil_div(resident, strips)));
    hipLaunchKernelGGL(kernel, dim3(strips, (unsigned)units), dim3(kF32Waves * 64), 0, st, g);
  };
  mark(1);
  // one block: four groups in flight, or two and twice the workgroups per CU where those are many and short
  if (blocks == 3) launch(gemm_f32_direct_kernel<true, 3, 2, 2>, 3, 512, g1);
  else if (s->d < 512 && (int64_t)dv.E_loc * ceil_div(s->f, 32) >= 768) launch(gemm_f32_direct_kernel<true, 1, 2, 4>, 1, 512, g1);
  else launch(gemm_f32_direct_kernel<true, 1, 4, 2>, 1, 512, g1);
  const int rc = launch_status();
  mark(2);
  if (rc != MOE_OK) return rc;
  launch(gemm_f32_direct_kernel<false, 1, 4, 4>, 1, 1024, g2);
  mark(3);
  return launch_status();
}

static int launch_combine(const moe_shape *s, const Derived &dv, const float *rows, const int32_t *topk_idx,
                          const moe_dispatch *tb, void *y, bool skip_sole, hipStream_t st) {
  const dim3 grid((unsigned)ceil_div(s->T, kCombineWaves)), block(kCombineWaves * 64);
#define MOE355_COMBINE(T_, FUSED_)                                                                             \
  hipLaunchKernelGGL((combine_kernel<T_, FUSED_>), grid, block, 0, st, rows, topk_idx, tb->inv_perm, tb->offsets, \
                     s->T, s->k, s->d, dv.e_lo, dv.E_loc, (int)dv.P_cap, static_cast<T_ *>(y))
  if (s->dtype == MOE_BF16) {
    if (skip_sole) MOE355_COMBINE(bf16_t, true); else MOE355_COMBINE(bf16_t, false);
  } else {
    if (skip_sole) MOE355_COMBINE(float, true); else MOE355_COMBINE(float, false);
  }
#undef MOE355_COMBINE
  return launch_status();
}

// Small batches: the stream kernels (stream_gemm.h).  The reduction ranges have to give each of the eight waves work
// (d, f >= 512).  A workgroup reads its expert's rows once per 32 columns, and an expert's weights once per 64 rows.
//   At most 12 rows per expert on average: always (2.3 GB of weights, 8 rows: 1.23 to 1.5 x the tile kernels' speed; 16, 24
//   and 32 rows of a 2.8 GB layer: 0.99, 0.91 and 0.81 x).
//   More rows: layers of at most 128 MB, where the launches saved count.  While an expert's rows fit one pass (T <= 64, or
//   48 rows on average) that holds for all of them (1.2 to 2.5 x at 16 to 64 rows).
//   Beyond, by estimated time (microseconds): the stream kernels take 4.6 (FP8: 4.0) per million weights of a matrix, the
//   tile kernels 30 (FP8: 38) and 0.88 per k-step of the two reductions.  Measured at 96 and 128 rows, tile time / stream time: 8
//   experts of 1024 x 1024 1.32 and 1.21 (FP8 1.45 and 1.30), 1536 x 1024 1.23 and 1.14 (1.31 and 1.20), 2048 x 1024 1.13 and
//   1.04 (0.93 and 0.83), 1536 x 1536 0.92 and 0.84 (1.04 and 0.91), 2048 x 1280 0.83 and 0.77 (0.94 and 0.85); 4 of 2048 x
//   2048 1.29 and 1.22 (1.02 and 0.92); 2 of 4096 x 2048 1.25 and 1.17 (1.33 and 1.26).
bool stream_form(const moe_shape *s, const Derived &dv, int elt) {
  if (s->dtype != MOE_BF16 || s->T > kStreamTokens || dv.E_loc > kStreamExperts || s->d < 512 || s->f < 512 ||
      stream2_lds_bytes(s->T, (int)dv.P_cap, dv.E_loc) > 160 * 1024)
    return false;
  // 32-bit offsets into the rows (2 GiB) and into one packed panel of 256 columns (512 bytes per reduction index)
  const int64_t widest = std::max(s->d, s->f);
  if (std::max<int64_t>(s->T, dv.P_cap) * widest * elt >= (int64_t)1 << 31 || widest >= 1 << 22) return false;
  const int64_t pairs = (int64_t)s->T * s->k, weights = (int64_t)dv.E_loc * s->d * s->f;
  if (pairs <= 12 * (int64_t)s->E) return true;
  if (weights * 3 * elt > (int64_t)128 << 20) return false;
  if (s->T <= 64 || pairs <= 48 * (int64_t)s->E) return true;
  const double stream = (elt == 1 ? 4.0e-6 : 4.6e-6) * weights;
  return stream <= (elt == 1 ? 38.0 : 30.0) + 0.88 / 128 * elt * ((double)s->d + s->f);
}

// Work groups per strip of GEMM-2: one, unless so few strips of 32 columns exist that handing the sums over (~1.5 us) costs
// less than what the missing CUs would have pulled (a CU pulls ~36 GB/s here, the chip ~6.5 TB/s, i.e. what ~180 CUs pull).
// Within 6 % of the best count at 1 to 128 tokens on 8 experts of 512 x 2048, 1024 x 1024 and 2048 x 512, 16 of 2048 x 2048 and
// 32 of 2880 x 2880 (one group instead: up to 2.6 x as long, 128 tokens of the first).
static int stream_groups(const moe_shape *s, const Derived &dv, int elt) {
  const int strips = ceil_div(s->d, 32);
  const double busy = std::min<double>(dv.E_loc, (double)s->T * s->k * dv.E_loc / s->E);
  const double us = busy * s->f * s->d * elt / 36e3;  // one CU, microseconds
  int best = 1;
  double t_best = us / std::min(strips, 180);
  for (int g = 2; g <= std::min(kStreamGroups, std::min(s->k, dv.E_loc)); ++g) {  // (the partial sums live in the rows of o)
    const double t = us / std::min(strips * g, 180) + 1.5;
    if (t < t_best) {
      t_best = t;
      best = g;
    }
  }
  return best;
}

static int launch_stream(const moe_shape *s, const Derived &dv, const void *x, const float *topk_w,
                         const moe_dispatch *tb, const void *packed_gu, const void *packed_down, const Ws &w, void *y,
                         hipStream_t st, void *const *events, const Fp8Operands *q) {
  auto mark = [&](int i) {
    if (events && events[i]) (void)hipEventRecord((hipEvent_t)events[i], st);
  };
  StreamArgs g1{};
  g1.A = q ? static_cast<const void *>(q->xq) : x;
  g1.Bp = packed_gu; g1.out = w.h;
  g1.offsets = tb->offsets; g1.perm = tb->perm; g1.topk_w = topk_w; g1.error = w.header + 24;
  g1.T = s->T; g1.k = s->k; g1.e_lo = dv.e_lo; g1.E_loc = dv.E_loc; g1.P_cap = (int)dv.P_cap;
  const int step = q ? kFp8KStep : kBK;
  g1.K = s->d; g1.N = s->f; g1.n_ntiles = ceil_div(s->f, kBN / 2); g1.n_ktiles = ceil_div(s->d, step);
  StreamArgs g2 = g1;
  const int groups = stream_groups(s, dv, q ? 1 : 2);
  g2.A = w.h; g2.Bp = packed_down; g2.out = y;
  g1.arrived = g2.arrived = w.arrived;
  g1.n_arrived = groups > 1 ? ceil_div(s->d, 32) : 0;
  g2.partial = w.o;
  g2.K = s->f; g2.N = s->d; g2.n_ntiles = ceil_div(s->d, kBN); g2.n_ktiles = ceil_div(s->f, step);
  if (q) {
    g1.a_scale = q->x_scale; g1.b_scale = q->gu_scale; g1.h_scale = q->h_scale;
    g2.b_scale = q->down_scale; g2.h_scale = q->h_scale;
  }
  mark(1);
  const dim3 grid1((unsigned)ceil_div(s->f, 32), (unsigned)dv.E_loc), grid2((unsigned)ceil_div(s->d, 32), (unsigned)groups);
  const size_t lds = stream2_lds_bytes(s->T, (int)dv.P_cap, dv.E_loc);
#define MOE355_STREAM(FP8_, NB_)                                                                            \
  do {                                                                                                                \
    static std::atomic<uint64_t> done{0};                                                                             \
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&stream_gemm2_kernel<FP8_, NB_>), 160 * 1024, done))    \
      return MOE_ERR_HIP;                                                                                             \
    hipLaunchKernelGGL((stream_gemm1_kernel<FP8_, NB_>), grid1, dim3(kStreamWaves * 64), 0, st, g1);                     \
    mark(2);                                                                                                          \
    hipLaunchKernelGGL((stream_gemm2_kernel<FP8_, NB_>), grid2, dim3(kStreamWaves * 64), lds, st, g2);          \
  } while (0)
  if (q) {
    if (stream_row_blocks(s->T) == 1) MOE355_STREAM(true, 1); else MOE355_STREAM(true, 2);
  } else {
    if (stream_row_blocks(s->T) == 1) MOE355_STREAM(false, 1); else MOE355_STREAM(false, 2);
  }
#undef MOE355_STREAM
  mark(3);
  mark(4);
  return launch_status();
}

static bool tables_ok(const moe_dispatch *t) {
  return t && t->counts && t->offsets && t->perm && t->inv_perm && t->rank_counts && t->rank_offsets &&
         t->dedup_tok && t->dedup_mask && t->pair_to_dedup;
}

}  // namespace moe355

using namespace moe355;

extern "C" int moe_pack_weights(const moe_shape *shape, const void *W_gate, const void *W_up, const void *W_down,
                                void *packed_gate_up, void *packed_down, void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!W_gate || !W_up || !W_down || !packed_gate_up || !packed_down) return MOE_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  begin_launches();
  const int d = shape->d, f = shape->f;
  if (shape->dtype == MOE_F32) {
    const size_t one = (size_t)dv.E_loc * d * f;
    float *gu = static_cast<float *>(packed_gate_up);
    hipLaunchKernelGGL(copy_f32_kernel, dim3(1024), dim3(256), 0, st, static_cast<const float *>(W_gate), gu, one);
    hipLaunchKernelGGL(copy_f32_kernel, dim3(1024), dim3(256), 0, st, static_cast<const float *>(W_up), gu + one, one);
    hipLaunchKernelGGL(copy_f32_kernel, dim3(1024), dim3(256), 0, st, static_cast<const float *>(W_down),
                       static_cast<float *>(packed_down), one);
    return launch_status();
  }
  const int nt1 = ceil_div(f, kBN / 2), kt1 = ceil_div(d, kBK);
  const int nt2 = ceil_div(d, kBN), kt2 = ceil_div(f, kBK);
  if (nt1 > 65535 || nt2 > 65535 || dv.E_loc > 65535) return MOE_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(pack_bf16_kernel<true>, dim3(kt1, nt1, dv.E_loc), dim3(256), 0, st,
                     static_cast<const bf16_t *>(W_gate), static_cast<const bf16_t *>(W_up),
                     static_cast<bf16_t *>(packed_gate_up), d, f, nt1, kt1);
  if ((rc = launch_status()) != MOE_OK) return rc;
  hipLaunchKernelGGL(pack_bf16_kernel<false>, dim3(kt2, nt2, dv.E_loc), dim3(256), 0, st,
                     static_cast<const bf16_t *>(W_down), static_cast<const bf16_t *>(nullptr),
                     static_cast<bf16_t *>(packed_down), f, d, nt2, kt2);
  return launch_status();
}

static int forward_common(const moe_shape *shape, const void *x, const int32_t *topk_idx, const float *topk_w,
                          const moe_dispatch *tables, const void *packed_gate_up, const void *packed_down, void *y,
                          void *workspace, size_t workspace_bytes, void *stream, bool fused,
                          void *const *events = nullptr, int gemm_launches = 0, const float *h_scale = nullptr,
                          void *keep = nullptr, int max_polls = kMaxPolls, int wait_extra = 0) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!x || !topk_idx || !topk_w || !packed_gate_up || !packed_down || !y || !tables_ok(tables))
    return MOE_ERR_INVALID_ARG;
  const bool fp8 = h_scale != nullptr;  // FP8 GEMMs: bf16 layers whose rows are whole 16-code chunks
  if (fp8 && (shape->dtype != MOE_BF16 || shape->d % 16 != 0 || shape->f % 16 != 0)) return MOE_ERR_UNSUPPORTED;
  const size_t need = fp8     ? moe_fp8_forward_workspace_bytes(shape)
                      : fused ? moe_forward_workspace_bytes(shape)
                              : moe_unfused_workspace_bytes(shape);
  if (!workspace || workspace_bytes < need) return MOE_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return MOE_ERR_INVALID_ARG;
  // rows are moved 16 bytes at a time
  if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(packed_gate_up) |
       reinterpret_cast<uintptr_t>(packed_down)) % 16 != 0)
    return MOE_ERR_INVALID_ARG;
  if ((int64_t)dv.max_mtiles * std::max(dv.nt1, dv.nt2) > (int64_t)1 << 30) return MOE_ERR_UNSUPPORTED;
  // gemm_launches: 0 = by shape, 1 = resident kernel with the tile-level hand-over (bf16 only), 2 = two launches,
  // 3 = resident kernel that also runs Combine (bf16 inference forward only)
  if ((gemm_launches == 1 || gemm_launches == 3) && shape->dtype != MOE_BF16) return MOE_ERR_UNSUPPORTED;
  const bool with_combine = gemm_launches == 3;
  if (with_combine && (!fused || fp8 || keep)) return MOE_ERR_UNSUPPORTED;
  if (with_combine && dv.E_loc > 4091) return MOE_ERR_UNSUPPORTED;  // (documented bound of this form)
  const bool pipelined = with_combine || (gemm_launches ? gemm_launches : tile_gemm_launches(shape, fp8 ? 1 : 2)) == 1;
  // a work item packs its N tile and its M-tile id into one word
  if (std::max(dv.nt1, dv.nt2) >= 1 << kTileShift || dv.max_mtiles >= 1 << (31 - kTileShift)) return MOE_ERR_UNSUPPORTED;
  // the GEMM kernels address A rows with 32-bit element offsets (row * row length)
  if (std::max<int64_t>(shape->T, dv.P_cap) * std::max(shape->d, shape->f) >= (int64_t)1 << 32) return MOE_ERR_UNSUPPORTED;
  if (shape->T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  begin_launches();
  const FwdLayout L = forward_layout(shape, dv);
  const Ws w = carve(workspace, L);
  auto mark = [&](int i) {
    if (events && events[i]) (void)hipEventRecord((hipEvent_t)events[i], st);
  };
  // fused bf16 layers: GEMM-2 writes the rows that need no reduction straight to y and Combine skips them.  The training
  // forward, which keeps every weighted row for the backward pass, does both: two more bytes written per element instead of
  // four read back.
  int32_t *sole = fused && shape->dtype == MOE_BF16 ? w.row_sole : nullptr;
  void *keep_gu = nullptr;
  float *keep_o = nullptr;
  if (keep) {
    const size_t rows = (size_t)(dv.P_cap > 0 ? dv.P_cap : 1);
    keep_gu = keep;
    keep_o = reinterpret_cast<float *>(static_cast<unsigned char *>(keep) + align_up(rows * 2 * shape->f * 2, 256));
  }
  mark(0);
  Fp8Operands q{};
  const bool streams = fused && !keep && gemm_launches == 0 && stream_form(shape, dv, fp8 ? 1 : 2);
  TokenCodes tokens{};
  if (fp8) {
    // x as codes with one scale per token, behind the tile-table part of the workspace
    unsigned char *b = static_cast<unsigned char *>(workspace);
    uint8_t *xq = b + L.total;
    float *x_scale = reinterpret_cast<float *>(b + L.total + align_up((size_t)shape->T * shape->d, 256));
    if (!streams && codes_with_table(shape, dv)) {
      tokens.x = static_cast<const uint4 *>(x);
      tokens.cols = shape->d;
      tokens.codes = xq;
      tokens.scales = x_scale;
      tokens.inv_perm = tables->inv_perm;
    } else {
      hipLaunchKernelGGL(fp8_quantize_rows_kernel, dim3((unsigned)shape->T), dim3(256), 0, st,
                         static_cast<const uint4 *>(x), shape->d, xq, x_scale);
      if ((rc = launch_status()) != MOE_OK) return rc;
    }
    q.xq = xq;
    q.x_scale = x_scale;
    q.gu_scale = reinterpret_cast<const float *>(static_cast<const unsigned char *>(packed_gate_up) +
                                                 align_up(fp8_tile_bytes(shape, dv, 0), 256));
    q.down_scale = reinterpret_cast<const float *>(static_cast<const unsigned char *>(packed_down) +
                                                   align_up(fp8_tile_bytes(shape, dv, 1), 256));
    q.h_scale = h_scale;
  }
  // the stream kernels are the form the library picks for a small batch; the forms a caller asks for by name (and the
  // training forward, which keeps its rows) run the tile kernels
  if (streams)
    return launch_stream(shape, dv, x, topk_w, tables, packed_gate_up, packed_down, w, y, st, events, fp8 ? &q : nullptr);
  if (const int blocks = fused && gemm_launches == 0 ? f32_direct_blocks(shape, dv) : 0) {
    if ((rc = launch_f32_direct(shape, dv, blocks, x, topk_w, tables, packed_gate_up, packed_down, w, st, events)) !=
        MOE_OK)
      return rc;
    rc = launch_combine(shape, dv, w.o, topk_idx, tables, y, false, st);
    mark(4);
    return rc;
  }
  if ((rc = launch_prep(shape, dv, tables, topk_idx, topk_w, w, sole, st, with_combine, tokens)) != MOE_OK) return rc;
  mark(1);
  if (fused) {
    if ((rc = launch_gemms(shape, dv, x, w.row_tok, shape->d, packed_gate_up, packed_down, w, sole, y, st,
                           events, pipelined, fp8 ? &q : nullptr, keep_gu, keep_o, max_polls, wait_extra,
                           with_combine ? tables : nullptr, topk_idx)) != MOE_OK)
      return rc;
    if (!with_combine) rc = launch_combine(shape, dv, keep ? keep_o : w.o, topk_idx, tables, y, sole != nullptr, st);
    mark(4);
    return rc;
  }
  // unfused: gather copy -> GEMMs on the copy -> zero -> atomic scatter-add -> cast
  unsigned char *b = static_cast<unsigned char *>(workspace);
  const size_t rows = (size_t)(dv.P_cap > 0 ? dv.P_cap : 1);
  void *xs = b + L.total;
  float *y32 = reinterpret_cast<float *>(b + L.total + align_up(rows * (size_t)shape->d * dv.elt, 256));
  const int row_chunks = shape->d * dv.elt / 16;
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)rows), dim3(256), 0, st, static_cast<const uint4 *>(x),
                     w.header, w.row_tok, row_chunks, static_cast<uint4 *>(xs));
  if ((rc = launch_status()) != MOE_OK) return rc;
  if ((rc = launch_gemms(shape, dv, xs, nullptr, shape->d, packed_gate_up, packed_down, w, nullptr, nullptr, st, nullptr,
                         pipelined)) != MOE_OK) return rc;
  const size_t n = (size_t)shape->T * shape->d;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(2048), dim3(256), 0, st, reinterpret_cast<float4 *>(y32), n / 4);
  hipLaunchKernelGGL(scatter_add_kernel, dim3((unsigned)rows), dim3(256), 0, st, w.o, w.header, w.row_tok, shape->d,
                     y32);
  if (shape->dtype == MOE_BF16)
    hipLaunchKernelGGL(cast_rows_kernel<bf16_t>, dim3(2048), dim3(256), 0, st, y32, static_cast<bf16_t *>(y), n / 8);
  else
    hipLaunchKernelGGL(cast_rows_kernel<float>, dim3(2048), dim3(256), 0, st, y32, static_cast<float *>(y), n / 8);
  return launch_status();
}

extern "C" size_t moe_fp8_packed_weight_bytes(const moe_shape *shape, int which) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK || (which != 0 && which != 1)) return 0;
  const size_t scales = (size_t)dv.E_loc * (which == 0 ? 2 * (size_t)shape->f : (size_t)shape->d) * sizeof(float);
  return align_up(fp8_tile_bytes(shape, dv, which), 256) + align_up(scales, 256);
}

extern "C" size_t moe_fp8_forward_workspace_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  const size_t T = (size_t)(shape->T > 0 ? shape->T : 1);
  return forward_layout(shape, dv).total + align_up(T * shape->d, 256) + align_up(T * sizeof(float), 256);
}

extern "C" int moe_fp8_pack_weights(const moe_shape *shape, const void *W_gate, const void *W_up, const void *W_down,
                                    void *packed_gate_up, void *packed_down, void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!W_gate || !W_up || !W_down || !packed_gate_up || !packed_down) return MOE_ERR_INVALID_ARG;
  if (shape->dtype != MOE_BF16 || shape->d % 16 != 0 || shape->f % 16 != 0) return MOE_ERR_UNSUPPORTED;
  if ((reinterpret_cast<uintptr_t>(packed_gate_up) | reinterpret_cast<uintptr_t>(packed_down)) % 16 != 0)
    return MOE_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  begin_launches();
  const int d = shape->d, f = shape->f;
  const int nt1 = ceil_div(f, kBN / 2), kt1 = ceil_div(d, kFp8KStep);
  const int nt2 = ceil_div(d, kBN), kt2 = ceil_div(f, kFp8KStep);
  if (nt1 > 65535 || nt2 > 65535 || dv.E_loc > 65535) return MOE_ERR_UNSUPPORTED;
  uint8_t *gu = static_cast<uint8_t *>(packed_gate_up), *dn = static_cast<uint8_t *>(packed_down);
  float *s_gu = reinterpret_cast<float *>(gu + align_up(fp8_tile_bytes(shape, dv, 0), 256));  // [E_loc][2][f]
  float *s_dn = reinterpret_cast<float *>(dn + align_up(fp8_tile_bytes(shape, dv, 1), 256));  // [E_loc][d]
  const bf16_t *Wg = static_cast<const bf16_t *>(W_gate), *Wu = static_cast<const bf16_t *>(W_up);
  const bf16_t *Wd = static_cast<const bf16_t *>(W_down);
  // column maxima (the reduction range cut into slices for enough workgroups), then scales in place
  const size_t n_gu = (size_t)dv.E_loc * 2 * f, n_dn = (size_t)dv.E_loc * d;
  hipLaunchKernelGGL(fill_f32_kernel, dim3(256), dim3(256), 0, st, s_gu, n_gu, 0.0f);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(256), dim3(256), 0, st, s_dn, n_dn, 0.0f);
  const int slices_d = std::max(1, std::min(32, d / 64)), slices_f = std::max(1, std::min(32, f / 64));
  hipLaunchKernelGGL(fp8_column_amax_kernel, dim3(ceil_div(f, 256), dv.E_loc, slices_d), dim3(256), 0, st, Wg, d, f,
                     reinterpret_cast<uint32_t *>(s_gu), 2 * f);
  hipLaunchKernelGGL(fp8_column_amax_kernel, dim3(ceil_div(f, 256), dv.E_loc, slices_d), dim3(256), 0, st, Wu, d, f,
                     reinterpret_cast<uint32_t *>(s_gu + f), 2 * f);
  hipLaunchKernelGGL(fp8_column_amax_kernel, dim3(ceil_div(d, 256), dv.E_loc, slices_f), dim3(256), 0, st, Wd, f, d,
                     reinterpret_cast<uint32_t *>(s_dn), d);
  hipLaunchKernelGGL(fp8_scales_from_amax_kernel, dim3(256), dim3(256), 0, st, s_gu, n_gu);
  hipLaunchKernelGGL(fp8_scales_from_amax_kernel, dim3(256), dim3(256), 0, st, s_dn, n_dn);
  if ((rc = launch_status()) != MOE_OK) return rc;
  hipLaunchKernelGGL(pack_fp8_kernel<true>, dim3(kt1, nt1, dv.E_loc), dim3(256), 0, st, Wg, Wu, s_gu, s_gu + f, 2 * f,
                     gu, d, f, nt1, kt1);
  if ((rc = launch_status()) != MOE_OK) return rc;
  hipLaunchKernelGGL(pack_fp8_kernel<false>, dim3(kt2, nt2, dv.E_loc), dim3(256), 0, st, Wd,
                     static_cast<const bf16_t *>(nullptr), s_dn, static_cast<const float *>(nullptr), d, dn, f, d, nt2,
                     kt2);
  return launch_status();
}

extern "C" int moe_fp8_quantize_rows(int64_t rows, int cols, const void *x, void *codes, float *scales,
                                     void *stream) {
  if (rows < 0 || rows > 0x7FFFFFFF || cols < 8 || cols % 8 != 0) return MOE_ERR_INVALID_ARG;
  if (!x || !codes || !scales) return MOE_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(x) % 16) != 0 || (reinterpret_cast<uintptr_t>(codes) % 8) != 0)
    return MOE_ERR_INVALID_ARG;
  if (rows == 0) return MOE_OK;
  begin_launches();
  hipLaunchKernelGGL(fp8_quantize_rows_kernel, dim3((unsigned)rows), dim3(256), 0, (hipStream_t)stream,
                     static_cast<const uint4 *>(x), cols, static_cast<uint8_t *>(codes), scales);
  return launch_status();
}

extern "C" int moe_fp8_fused_forward(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                     const float *topk_w, const moe_dispatch *tables, const void *packed_gate_up,
                                     const void *packed_down, const float *h_scale, void *y, void *workspace,
                                     size_t workspace_bytes, void *stream, void *const *events) {
  if (!h_scale) return MOE_ERR_INVALID_ARG;
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true, events, 0, h_scale);
}

extern "C" int moe_fused_forward(const moe_shape *shape, const void *x, const int32_t *topk_idx, const float *topk_w,
                                 const moe_dispatch *tables, const void *packed_gate_up, const void *packed_down,
                                 void *y, void *workspace, size_t workspace_bytes, void *stream) {
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true);
}

extern "C" int moe_fused_forward_bounded(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                         const float *topk_w, const moe_dispatch *tables, const void *packed_gate_up,
                                         const void *packed_down, void *y, void *workspace, size_t workspace_bytes,
                                         void *stream, int max_polls, int wait_extra) {
  if (max_polls < 1 || wait_extra < 0) return MOE_ERR_INVALID_ARG;
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true, nullptr, 1, nullptr, nullptr, max_polls, wait_extra);
}

extern "C" int moe_forward_status(const void *workspace, int32_t *flag, void *stream) {
  if (!workspace || !flag) return MOE_ERR_INVALID_ARG;
  // header word 24 of the forward workspace (see FwdLayout): raised by a wait of the resident kernel that gave up
  const int32_t *word = static_cast<const int32_t *>(workspace) + 24;
  hipStream_t st = (hipStream_t)stream;
  if (hipMemcpyAsync(flag, word, sizeof(int32_t), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess) {
    (void)hipGetLastError();
    return MOE_ERR_HIP;
  }
  return MOE_OK;
}

extern "C" int moe_fused_forward_timed(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                       const float *topk_w, const moe_dispatch *tables, const void *packed_gate_up,
                                       const void *packed_down, void *y, void *workspace, size_t workspace_bytes,
                                       void *stream, void *const *events) {
  if (!events) return MOE_ERR_INVALID_ARG;
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true, events);
}

extern "C" int moe_fused_forward_two_launch(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                            const float *topk_w, const moe_dispatch *tables,
                                            const void *packed_gate_up, const void *packed_down, void *y,
                                            void *workspace, size_t workspace_bytes, void *stream,
                                            void *const *events) {
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true, events, 2);
}

extern "C" int moe_fused_forward_one_launch(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                            const float *topk_w, const moe_dispatch *tables,
                                            const void *packed_gate_up, const void *packed_down, void *y,
                                            void *workspace, size_t workspace_bytes, void *stream,
                                            void *const *events) {
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true, events, 1);
}

extern "C" int moe_fused_forward_resident(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                          const float *topk_w, const moe_dispatch *tables, const void *packed_gate_up,
                                          const void *packed_down, void *y, void *workspace, size_t workspace_bytes,
                                          void *stream, void *const *events, int max_polls, int wait_extra) {
  if (max_polls < 0 || wait_extra < 0) return MOE_ERR_INVALID_ARG;
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true, events, 3, nullptr, nullptr, max_polls ? max_polls : kMaxPolls,
                        wait_extra);
}

extern "C" int moe_unfused_forward(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                   const float *topk_w, const moe_dispatch *tables, const void *packed_gate_up,
                                   const void *packed_down, void *y, void *workspace, size_t workspace_bytes,
                                   void *stream) {
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, false);
}

// ------------------------------------------------------------------------------------------------
// Training path: forward that keeps what the backward pass needs, and the backward pass.
// ------------------------------------------------------------------------------------------------
namespace moe355 {

// Backward workspace: the tile table (lists for the two backward GEMMs), the per-row metadata and the intermediates.
struct BwdLayout {
  FwdLayout t;   // header .. tile_ready as in the forward layout (h and o unused)
  size_t dgu;    // bf16 [P_cap, 2 f]  dg, then du
  size_t hw;     // bf16 [P_cap, f]    w silu(g) u
  size_t dxr;    // float[P_cap, d]    rows of dx before the per-token sum
  // weight gradients: operands transposed to [64-row block][column][64 rows], every expert's rows padded to blocks
  size_t kb;     // int32[E_loc + 1]   first block of every local expert in the padded row order
  size_t xT, dyT;  // bf16 [blocks][d][64]   gathered x rows, gathered dy rows
  size_t hwT;    // bf16 [blocks][f][64]
  size_t dguT;   // bf16 [blocks][2 f][64]
  size_t kpad;   // padded row capacity: 64 (ceil(P_cap / 64) + E_loc)
  size_t total;
};

static Derived backward_derived(const moe_shape *s, const Derived &dv) {
  Derived b = dv;
  b.nt1 = ceil_div(s->f, kBN);  // first backward GEMM: dh over f in plain 256-column tiles
  return b;
}

static BwdLayout backward_layout(const moe_shape *s, const Derived &dvb) {
  BwdLayout L;
  size_t off = 0;
  auto take = [&off](size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes, 256);
    return at;
  };
  const size_t rows = (size_t)(dvb.P_cap > 0 ? dvb.P_cap : 1);
  L.t.header = take(32 * sizeof(int32_t));
  L.t.tickets = take(16 * kTicketStride * sizeof(int32_t));
  L.t.work1 = take((size_t)dvb.max_mtiles * dvb.nt1 * 4 * sizeof(int32_t));
  L.t.work2 = take((size_t)dvb.max_mtiles * dvb.nt2 * 4 * sizeof(int32_t));
  L.t.row_tok = take(rows * sizeof(int32_t));
  L.t.row_w = take(rows * sizeof(float));
  L.t.row_sole = take(rows * sizeof(int32_t));
  L.t.tile_ready = take((size_t)dvb.max_mtiles * kReadyStride * sizeof(int32_t));
  L.t.row_tile = L.t.tile_done = L.t.arrived = 0;  // forward only
  L.t.h = L.t.o = 0;
  L.dgu = take(rows * 2 * (size_t)s->f * 2);
  L.hw = take(rows * (size_t)s->f * 2);
  L.dxr = take(rows * (size_t)s->d * sizeof(float));
  L.kpad = 64 * ((rows + 63) / 64 + (size_t)dvb.E_loc);
  L.kb = take((size_t)(dvb.E_loc + 1) * sizeof(int32_t));
  L.xT = take((size_t)s->d * L.kpad * 2);
  L.dyT = take((size_t)s->d * L.kpad * 2);
  L.hwT = take((size_t)s->f * L.kpad * 2);
  L.dguT = take(2 * (size_t)s->f * L.kpad * 2);
  L.t.total = L.total = off;
  return L;
}

// The two backward GEMMs as one resident launch, where they take 0.1 ms and more (estimated from the weights' bytes and from the
// flops).  Time of the backward pass without weight gradients in one launch over two, by rows per expert (even load / training
// load spread / power law):
//                               64              76 to 120       150 to 260      300 to 450      500 to 575
//   16 of 128 of 4096 x 1536    1.10 1.08 1.02  0.94 0.98 0.93  0.96 0.91 0.99  1.01 0.99 0.91  0.94 0.98 0.90
//   16 of 128 of 4096 x 1024    < 0.1 ms        < 0.1 ms        < 0.1 ms        1.02 1.00 1.00  1.02 1.00 0.99
//   16 of 128 of 7168 x 1024    1.02 1.00 0.93  0.96 0.95 0.95  0.97 0.91 0.96  0.97 0.96 0.96  0.99 0.98 0.91
//   16 of 32 of 4096 x 2048     0.98 1.10 0.89  0.93 0.96 0.89  0.97 0.91 0.92  1.02 0.93 0.88  0.89 0.90 0.97
//   32 of 128 of 2880 x 2880    0.93 0.96 0.89  0.91 0.90 0.92  0.90 0.94 0.95  1.01 0.94 0.99  0.99 1.00 1.00
//   32 of 256 of 7168 x 2048    0.96 0.96 0.96  0.91 0.92 0.94  0.96 0.89 0.93  1.00 0.95 0.95  0.97 0.96 0.97
//   64 of 2048 x 1024           0.94 0.93 0.93  0.90 0.91 0.93  0.94 0.90 0.90  0.98 0.92 0.93  0.97 0.95 0.96
//   8 of 64 of 8192 x 2048      0.98 0.97 0.92  0.95 0.96 0.95  0.95 0.90 1.00  1.01 0.95 0.94  1.02 0.99 0.92
//   8 of 64 of 4096 x 4096      -               0.99 0.98 1.03  0.96 0.94 0.99  1.02 0.98 0.89  0.90 0.88 1.02
//   8 of 4096 x 14336           0.97 0.96 0.94  1.02 1.00 0.97  1.03 1.00 0.96  1.01 1.01 0.99  0.99 0.99 0.96
//   4 of 8 of 4096 x 14336      -               0.97 0.98 0.95  0.99 0.99 1.03  1.03 1.01 1.02  1.04 1.01 0.97
//   8 of 32 of 2048 x 4096      < 0.1 ms        < 0.1 ms        < 0.1 ms        1.05 0.99 1.03  1.01 1.04 0.96
// Around 64 rows, where some experts have a tile of 64 rows and others one of 128, it pays from 32 experts on.  The second GEMM needs an item
// per CU in every M tile's share of experts: with fewer its last round is nearly empty in either form and the rows of [dg | du] past
// the L2s are all that differs (4096 x 14336, 2048 x 4096); half as many do where an expert has three M tiles.  From 600 rows on
// (750: 1.04, 2000: 1.02) those rows cost more than the last round of the first GEMM.  Below 0.1 ms: 8 of 64 of 2048 x 512 1.05 to 1.15.
static bool backward_one_launch(const moe_shape *s, const Derived &dv) {
  const double rows = (double)s->T * s->k / s->E, work = 3.0 * dv.E_loc * s->d * s->f;
  const int64_t items = (int64_t)dv.E_loc * ceil_div(s->d, kBN);  // of the second GEMM, per M tile of an expert
  return rows >= (dv.E_loc >= 32 ? 64 : 76) && rows < 600 && items >= (rows >= 512 ? 128 : 256) &&
         std::max(work * 2 / 6e12, 2 * rows * work / 1.1e15) >= 100e-6;
}

// Whether 32-bit offsets reach the operands of the two backward GEMMs (else: 64-bit ones, and two launches).
struct BwdFar { bool dy, dgu; };
static BwdFar backward_far(const moe_shape *s, const Derived &dv) {
  const int64_t end = (int64_t)1 << 32;
  return {(int64_t)s->T * s->d * 2 >= end, dv.P_cap * 2 * s->f * 2 >= end};
}

static bool backward_supported(const moe_shape *s) { return s->dtype == MOE_BF16 && s->f % kBK == 0; }

}  // namespace moe355

extern "C" int moe_backward_gemm_launches(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK || !backward_supported(shape)) return 0;
  const BwdFar far = backward_far(shape, dv);
  return !far.dy && !far.dgu && backward_one_launch(shape, dv) ? 1 : 2;
}

extern "C" size_t moe_train_kept_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  const size_t rows = (size_t)(dv.P_cap > 0 ? dv.P_cap : 1);
  return align_up(rows * 2 * shape->f * 2, 256) + align_up(rows * (size_t)shape->d * sizeof(float), 256);
}

extern "C" size_t moe_backward_workspace_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  return backward_layout(shape, backward_derived(shape, dv)).total;
}

extern "C" size_t moe_backward_packed_weight_bytes(const moe_shape *shape, int which) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK || (which != 0 && which != 1)) return 0;
  if (which == 0) return (size_t)dv.E_loc * ceil_div(shape->f, kBN) * ceil_div(shape->d, kBK) * kTileBytes;  // Wd^T
  return (size_t)dv.E_loc * ceil_div(shape->d, kBN) * (2 * ceil_div(shape->f, kBK)) * kTileBytes;  // [Wg^T; Wu^T]
}

extern "C" int moe_pack_weights_backward(const moe_shape *shape, const void *W_gate, const void *W_up,
                                         const void *W_down, void *packed_down_t, void *packed_gate_up_t,
                                         void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!W_gate || !W_up || !W_down || !packed_down_t || !packed_gate_up_t) return MOE_ERR_INVALID_ARG;
  if (!backward_supported(shape)) return MOE_ERR_UNSUPPORTED;
  if ((reinterpret_cast<uintptr_t>(W_gate) | reinterpret_cast<uintptr_t>(W_up) | reinterpret_cast<uintptr_t>(W_down) |
       reinterpret_cast<uintptr_t>(packed_down_t) | reinterpret_cast<uintptr_t>(packed_gate_up_t)) % 16 != 0)
    return MOE_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  begin_launches();
  const int d = shape->d, f = shape->f;
  const int ntf = ceil_div(f, kBN), ktd = ceil_div(d, kBK), ntd = ceil_div(d, kBN), ktf = f / kBK;
  if (ntf > 65535 || ntd > 65535 || dv.E_loc > 65535) return MOE_ERR_UNSUPPORTED;
  // B[k = model index][n = hidden index] = W_down[n][k]
  hipLaunchKernelGGL(pack_bf16_transposed_kernel, dim3(ktd, ntf, dv.E_loc), dim3(256), 0, st,
                     static_cast<const bf16_t *>(W_down), static_cast<bf16_t *>(packed_down_t), d, f, ntf, ktd, 0);
  // B[k = hidden index, gate then up][n = model index] = W_gate[n][k], W_up[n][k]
  hipLaunchKernelGGL(pack_bf16_transposed_kernel, dim3(ktf, ntd, dv.E_loc), dim3(256), 0, st,
                     static_cast<const bf16_t *>(W_gate), static_cast<bf16_t *>(packed_gate_up_t), f, d, ntd, 2 * ktf, 0);
  hipLaunchKernelGGL(pack_bf16_transposed_kernel, dim3(ktf, ntd, dv.E_loc), dim3(256), 0, st,
                     static_cast<const bf16_t *>(W_up), static_cast<bf16_t *>(packed_gate_up_t), f, d, ntd, 2 * ktf, ktf);
  return launch_status();
}

extern "C" int moe_fused_forward_train(const moe_shape *shape, const void *x, const int32_t *topk_idx,
                                       const float *topk_w, const moe_dispatch *tables, const void *packed_gate_up,
                                       const void *packed_down, void *y, void *kept, size_t kept_bytes,
                                       void *workspace, size_t workspace_bytes, void *stream) {
  if (!shape) return MOE_ERR_INVALID_ARG;
  if (shape->dtype != MOE_BF16) return MOE_ERR_UNSUPPORTED;
  if (!kept || kept_bytes < moe_train_kept_bytes(shape)) return MOE_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(kept) % 256 != 0) return MOE_ERR_INVALID_ARG;
  return forward_common(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace,
                        workspace_bytes, stream, true, nullptr, 0, nullptr, kept);
}

// Where the weight gradients come from transposed operands (4 GiB and more, or where a caller asks for it), the backward pass
// makes them beside its compute-bound GEMMs: those kernels need at most 16 registers and little or no LDS, so their waves fit
// on a CU next to a GEMM workgroup.  They go to a stream of the library's own (one per device, default priority, created on
// first use and kept), forked from and joined to the caller's stream by events.
struct SideStream {
  hipStream_t stream;
  hipEvent_t fork, mid, join;
  std::mutex enqueue;  // held by a call from its fork to its join: the events are re-recorded by every call
};
static SideStream *side_stream() {
  static SideStream made[64];  // (the mutex makes the struct non-trivial: default-constructed once)
  static std::atomic<int> state[64];  // 0 none, 1 being made, 2 ready
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  if (state[dev].load(std::memory_order_acquire) == 2) return &made[dev];
  int expect = 0;
  if (state[dev].compare_exchange_strong(expect, 1)) {
    SideStream &m = made[dev];
    if (hipStreamCreateWithFlags(&m.stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&m.fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&m.mid, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&m.join, hipEventDisableTiming) != hipSuccess) {
      state[dev].store(0);
      return nullptr;
    }
    state[dev].store(2, std::memory_order_release);
    return &m;
  }
  while (state[dev].load(std::memory_order_acquire) == 1) {
  }
  return state[dev].load(std::memory_order_acquire) == 2 ? &made[dev] : nullptr;
}

static int backward_common(const moe_shape *shape, const void *x, const void *dy, const int32_t *topk_idx,
                           const float *topk_w, const moe_dispatch *tables, const void *packed_down_t,
                           const void *packed_gate_up_t, const void *kept, size_t kept_bytes, void *dx, float *d_topk_w,
                           void *dW_gate, void *dW_up, void *dW_down, void *workspace, size_t workspace_bytes, void *stream,
                           bool copies, bool force_one_launch = false, int max_polls = kMaxPolls, int wait_extra = 0) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!x || !dy || !topk_idx || !topk_w || !packed_down_t || !packed_gate_up_t || !dx || !d_topk_w ||
      !tables_ok(tables))
    return MOE_ERR_INVALID_ARG;
  const bool wgrad = dW_gate || dW_up || dW_down;
  if (wgrad && !(dW_gate && dW_up && dW_down)) return MOE_ERR_INVALID_ARG;  // all three or none
  if (!backward_supported(shape)) return MOE_ERR_UNSUPPORTED;
  if (!kept || kept_bytes < moe_train_kept_bytes(shape)) return MOE_ERR_WORKSPACE;
  if (!workspace || workspace_bytes < moe_backward_workspace_bytes(shape)) return MOE_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(kept)) % 256 != 0)
    return MOE_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(dx) |
       reinterpret_cast<uintptr_t>(packed_down_t) | reinterpret_cast<uintptr_t>(packed_gate_up_t)) % 16 != 0)
    return MOE_ERR_INVALID_ARG;
  const Derived dvb = backward_derived(shape, dv);
  if ((int64_t)dvb.max_mtiles * std::max(dvb.nt1, dvb.nt2) > (int64_t)1 << 30) return MOE_ERR_UNSUPPORTED;
  if (std::max(dvb.nt1, dvb.nt2) >= 1 << kTileShift || dvb.max_mtiles >= 1 << (31 - kTileShift)) return MOE_ERR_UNSUPPORTED;
  if (std::max<int64_t>(shape->T, dv.P_cap) * std::max(shape->d, 2 * shape->f) >= (int64_t)1 << 32) return MOE_ERR_UNSUPPORTED;
  if (wgrad && (reinterpret_cast<uintptr_t>(dW_gate) | reinterpret_cast<uintptr_t>(dW_up) |
                reinterpret_cast<uintptr_t>(dW_down)) % 16 != 0)
    return MOE_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  begin_launches();
  const size_t n_pairs = (size_t)shape->T * shape->k;
  if (shape->T == 0) {
    if (wgrad) {  // no rows: every weight gradient is zero (bf16 zeros are zero words)
      const size_t words = (size_t)dv.E_loc * shape->d * shape->f / 2;
      for (void *p : {dW_gate, dW_up, dW_down})
        hipLaunchKernelGGL(fill_f32_kernel, dim3(1024), dim3(256), 0, st, static_cast<float *>(p), words, 0.0f);
    }
    return launch_status();
  }
  const BwdLayout L = backward_layout(shape, dvb);
  // weight gradients straight from the operands, where 32-bit offsets reach their rows and one behind the last token (row T:
  // the zeros behind an expert's rows); else, or where the caller asks for them, from transposed copies
  const int64_t reach = ((int64_t)1 << 32) - (1 << 16);
  const bool direct = !copies && std::max(((int64_t)shape->T + 1) * shape->d, dv.P_cap * 2 * shape->f) * 2 < reach;
  const auto tiles = [&](int edge) {  // of all three gradients of an expert
    const int64_t td = ceil_div(shape->d, edge);
    return td * ceil_div(2 * shape->f, edge) + td * ceil_div(shape->f, edge);
  };
  const BwdFar far = backward_far(shape, dv);
  if (force_one_launch && (far.dy || far.dgu || (wgrad && !direct))) return MOE_ERR_UNSUPPORTED;
  const int kblocks = (int)(L.kpad / 64);
  if (wgrad && (kblocks > 65535 || (direct && tiles(kBM) * dv.E_loc >= (int64_t)1 << 30))) return MOE_ERR_UNSUPPORTED;
  const Ws w = carve(workspace, L.t);
  unsigned char *b = static_cast<unsigned char *>(workspace);
  bf16_t *dgu = reinterpret_cast<bf16_t *>(b + L.dgu), *hw = reinterpret_cast<bf16_t *>(b + L.hw);
  float *dxr = reinterpret_cast<float *>(b + L.dxr);
  const size_t rows = (size_t)(dv.P_cap > 0 ? dv.P_cap : 1);
  const bf16_t *kept_gu = static_cast<const bf16_t *>(kept);
  const float *kept_o = reinterpret_cast<const float *>(static_cast<const unsigned char *>(kept) +
                                                        align_up(rows * 2 * shape->f * 2, 256));
  if ((rc = launch_prep(shape, dvb, tables, topk_idx, topk_w, w, w.row_sole, st)) != MOE_OK) return rc;
  // side stream (transposed operands): nothing on it reads a GEMM's output before `mid`
  SideStream *side = nullptr;
  std::unique_lock<std::mutex> side_lock;  // (released when the call returns)
  int32_t *kb = reinterpret_cast<int32_t *>(b + L.kb);
  bf16_t *xT = reinterpret_cast<bf16_t *>(b + L.xT), *dyT = reinterpret_cast<bf16_t *>(b + L.dyT);
  bf16_t *hwT = reinterpret_cast<bf16_t *>(b + L.hwT), *dguT = reinterpret_cast<bf16_t *>(b + L.dguT);
  const auto transpose = [&](const bf16_t *src, const int32_t *map, int ld, int C, bf16_t *dst) {
    hipLaunchKernelGGL(gather_transpose_kernel, dim3(ceil_div(C, 64), kblocks), dim3(256), 0, side->stream, src, map,
                       ld, 0, C, tables->offsets, w.header, kb, dv.e_lo, dv.E_loc, dst);
  };
  // from the fork on, every return first makes the caller's stream wait for the side stream
  const auto join = [&](int code) {
    if (!side) return code;
    if (hipEventRecord(side->join, side->stream) != hipSuccess || hipStreamWaitEvent(st, side->join, 0) != hipSuccess)
      return code != MOE_OK ? code : (int)MOE_ERR_HIP;
    return code;
  };
  if (wgrad && !direct) {
    if (!(side = side_stream())) return MOE_ERR_HIP;
    side_lock = std::unique_lock<std::mutex>(side->enqueue);
    if (hipEventRecord(side->fork, st) != hipSuccess || hipStreamWaitEvent(side->stream, side->fork, 0) != hipSuccess) {
      side = nullptr;
      return MOE_ERR_HIP;
    }
    hipLaunchKernelGGL(wgrad_blocks_kernel, dim3(1), dim3(256), 0, side->stream, tables->offsets, w.header, dv.e_lo,
                       dv.E_loc, kb);
    transpose(static_cast<const bf16_t *>(x), w.row_tok, shape->d, shape->d, xT);
    transpose(static_cast<const bf16_t *>(dy), w.row_tok, shape->d, shape->d, dyT);
    if ((rc = launch_status()) != MOE_OK) return join(rc);
  }
  hipLaunchKernelGGL(gate_weight_grad_kernel, dim3((unsigned)std::min<size_t>(4096, (rows + 3) / 4)), dim3(256), 0, st,
                     kept_o, static_cast<const bf16_t *>(dy), w.header, w.row_tok, w.row_w, tables->perm, tables->inv_perm,
                     (int)n_pairs, shape->d, d_topk_w);
  if ((rc = launch_status()) != MOE_OK) return join(rc);
  const auto grid_of = [&](int nt) { return dim3((unsigned)(((size_t)dvb.max_mtiles * nt + 255) / 256 * 256)); };
  // dh_raw = dy[token of the row] Wd^T, then the SwiGLU derivative with the kept g and u
  GemmArgs g1{};
  g1.A = dy; g1.row_map = w.row_tok; g1.Bp = packed_down_t; g1.out = dgu; g1.row_w = w.row_w;
  g1.aux = const_cast<bf16_t *>(kept_gu); g1.aux2 = hw;
  g1.n_items = w.header + 0; g1.work = w.work1;
  g1.K = shape->d; g1.N = shape->f; g1.lda = shape->d; g1.ldo = 2 * shape->f;
  g1.n_ntiles = dvb.nt1; g1.n_ktiles = ceil_div(shape->d, kBK);
  const bool one_launch = force_one_launch || (!side && !far.dy && !far.dgu && backward_one_launch(shape, dv));
  if (!one_launch) {
    rc = side ? launch_items<false, false, true, true>(g1, far.dy, grid_of(dvb.nt1), st)
              : launch_items<false, false, true, false>(g1, far.dy, grid_of(dvb.nt1), st);
    if (rc != MOE_OK) return join(rc);
  }
  if (side) {  // dg, du and w h are there: their transposes run beside the second GEMM
    if (hipEventRecord(side->mid, st) != hipSuccess || hipStreamWaitEvent(side->stream, side->mid, 0) != hipSuccess)
      return join(MOE_ERR_HIP);
    transpose(hw, nullptr, shape->f, shape->f, hwT);
    transpose(dgu, nullptr, 2 * shape->f, 2 * shape->f, dguT);
    if ((rc = launch_status()) != MOE_OK) return join(rc);
  }
  // rows of dx = [dg | du] [Wg^T ; Wu^T]; a row that is its token's only local slot goes straight to dx
  GemmArgs g2{};
  g2.A = dgu; g2.row_map = nullptr; g2.Bp = packed_gate_up_t; g2.out = dxr; g2.row_w = nullptr;
  g2.row_sole = w.row_sole; g2.y = dx;
  g2.n_items = w.header + 3; g2.work = w.work2;
  g2.K = 2 * shape->f; g2.N = shape->d; g2.lda = 2 * shape->f; g2.ldo = shape->d;
  g2.n_ntiles = dvb.nt2; g2.n_ktiles = 2 * (shape->f / kBK);
  if (one_launch) {
    PipelineArgs pa{};
    pa.g1 = g1; pa.g2 = g2;
    pa.tickets = w.tickets; pa.tile_ready = w.tile_ready; pa.error = w.header + 24;
    pa.nt1 = dvb.nt1 + wait_extra; pa.max_polls = max_polls;
    rc = launch_resident<gemm_backward_pipeline_kernel>(pa, st);
  } else {
    rc = side ? launch_items<false, false, false, true>(g2, far.dgu, grid_of(dvb.nt2), st)
              : launch_items<false, false, false, false>(g2, far.dgu, grid_of(dvb.nt2), st);
  }
  if (rc != MOE_OK) return join(rc);
  if ((rc = launch_combine(shape, dv, dxr, topk_idx, tables, dx, true, st)) != MOE_OK || !wgrad) return join(rc);
  if ((rc = join(MOE_OK)) != MOE_OK) return rc;
  if (direct) {
    WgradDirectArgs a;
    a.x = static_cast<const bf16_t *>(x); a.dy = static_cast<const bf16_t *>(dy); a.dgu = dgu; a.hw = hw;
    a.dW_gate = static_cast<bf16_t *>(dW_gate); a.dW_up = static_cast<bf16_t *>(dW_up);
    a.dW_down = static_cast<bf16_t *>(dW_down);
    a.offsets = tables->offsets; a.header = w.header; a.row_tok = w.row_tok;
    a.e_lo = dv.e_lo; a.E_loc = dv.E_loc; a.T = shape->T; a.d = shape->d; a.f = shape->f;
    a.n_items = (int)(tiles(kBM) * dv.E_loc);
    static std::atomic<uint64_t> done_d{0};
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&wgrad_bf16_kernel), kWgradLds, done_d)) return MOE_ERR_HIP;
    hipLaunchKernelGGL(wgrad_bf16_kernel, dim3((unsigned)align_up(a.n_items, 8 * kChunk)), dim3(kGemmThreads), kWgradLds, st,
                       a);
    if ((rc = launch_status()) != MOE_OK) return rc;
    hipLaunchKernelGGL(wgrad_thin_bf16_kernel, dim3((unsigned)(tiles(128) + kThinTiles - 1) / kThinTiles, dv.E_loc), dim3(256), 0,
                       st, a);
    return launch_status();
  }
  const size_t units = (size_t)shape->d * shape->f / 8;  // 16-byte units of one expert's gradient
  hipLaunchKernelGGL(wgrad_zero_empty_kernel,
                     dim3((unsigned)std::min<size_t>(1024, ceil_div(units, (size_t)8192)), dv.E_loc, 3), dim3(256), 0,
                     st, tables->offsets, w.header, dv.e_lo, static_cast<u32x4 *>(dW_gate), static_cast<u32x4 *>(dW_up),
                     static_cast<u32x4 *>(dW_down), units);
  // one grouped product per weight matrix, over the transposed operands
  static std::atomic<uint64_t> done_w{0};
  if (!allow_dynamic_lds(reinterpret_cast<const void *>(&wgrad_slab_kernel), 2 * kStageBytes, done_w)) return MOE_ERR_HIP;
  const auto product = [&](const bf16_t *AT, int lda, const bf16_t *BT, int ldb, int b0, int M, int N, void *C) {
    WgradArgs a;
    a.AT = AT; a.BT = BT; a.C = static_cast<bf16_t *>(C); a.kb = kb;
    a.lda = lda; a.ldb = ldb; a.a0 = 0; a.b0 = b0;
    a.M = M; a.N = N; a.n_mt = ceil_div(M, kBM); a.n_nt = ceil_div(N, kBN);
    hipLaunchKernelGGL(wgrad_slab_kernel, dim3(a.n_mt * a.n_nt, dv.E_loc), dim3(kGemmThreads), 2 * kStageBytes, st, a);
    a.n_mt = ceil_div(M, 128); a.n_nt = ceil_div(N, 128);  // experts with few or no rows: small tiles
    hipLaunchKernelGGL(wgrad_thin_slab_kernel, dim3(ceil_div(a.n_mt * a.n_nt, kThinTiles), dv.E_loc), dim3(256), 0, st,
                       a);
  };
  product(xT, shape->d, dguT, 2 * shape->f, 0, shape->d, shape->f, dW_gate);         // x^T dg
  product(xT, shape->d, dguT, 2 * shape->f, shape->f, shape->d, shape->f, dW_up);    // x^T du
  product(hwT, shape->f, dyT, shape->d, 0, shape->f, shape->d, dW_down);             // (w h)^T dy
  return launch_status();
}

extern "C" int moe_fused_backward(const moe_shape *shape, const void *x, const void *dy, const int32_t *topk_idx,
                                  const float *topk_w, const moe_dispatch *tables, const void *packed_down_t,
                                  const void *packed_gate_up_t, const void *kept, size_t kept_bytes, void *dx,
                                  float *d_topk_w, void *dW_gate, void *dW_up, void *dW_down, void *workspace,
                                  size_t workspace_bytes, void *stream) {
  return backward_common(shape, x, dy, topk_idx, topk_w, tables, packed_down_t, packed_gate_up_t, kept, kept_bytes, dx,
                         d_topk_w, dW_gate, dW_up, dW_down, workspace, workspace_bytes, stream, false);
}

extern "C" int moe_fused_backward_copies(const moe_shape *shape, const void *x, const void *dy, const int32_t *topk_idx,
                                         const float *topk_w, const moe_dispatch *tables, const void *packed_down_t,
                                         const void *packed_gate_up_t, const void *kept, size_t kept_bytes, void *dx,
                                         float *d_topk_w, void *dW_gate, void *dW_up, void *dW_down, void *workspace,
                                         size_t workspace_bytes, void *stream) {
  return backward_common(shape, x, dy, topk_idx, topk_w, tables, packed_down_t, packed_gate_up_t, kept, kept_bytes, dx,
                         d_topk_w, dW_gate, dW_up, dW_down, workspace, workspace_bytes, stream, true);
}

extern "C" int moe_fused_backward_bounded(const moe_shape *shape, const void *x, const void *dy, const int32_t *topk_idx,
                                          const float *topk_w, const moe_dispatch *tables, const void *packed_down_t,
                                          const void *packed_gate_up_t, const void *kept, size_t kept_bytes, void *dx,
                                          float *d_topk_w, void *dW_gate, void *dW_up, void *dW_down, void *workspace,
                                          size_t workspace_bytes, void *stream, int max_polls, int wait_extra) {
  if (max_polls < 1 || wait_extra < 0) return MOE_ERR_INVALID_ARG;
  return backward_common(shape, x, dy, topk_idx, topk_w, tables, packed_down_t, packed_gate_up_t, kept, kept_bytes, dx,
                         d_topk_w, dW_gate, dW_up, dW_down, workspace, workspace_bytes, stream, false, true, max_polls,
                         wait_extra);
}

extern "C" int moe_dispatch_gather(const moe_shape *shape, const void *x, const moe_dispatch *tables, void *xs,
                                   void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!x || !xs || !tables_ok(tables)) return MOE_ERR_INVALID_ARG;
  if (shape->T == 0) return MOE_OK;
  const int nlr = shape->local_rank_end - shape->local_rank_begin;
  const int64_t max_entries = (int64_t)shape->T * (shape->k < nlr ? shape->k : nlr);
  begin_launches();
  hipLaunchKernelGGL(dispatch_gather_kernel, dim3((unsigned)max_entries), dim3(256), 0, (hipStream_t)stream,
                     static_cast<const uint4 *>(x), tables->rank_offsets, tables->dedup_tok, tables->dedup_mask,
                     tables->inv_perm, tables->offsets, shape->T, shape->k, shape->local_rank_begin,
                     shape->local_rank_end, dv.e_lo, (int)dv.P_cap, shape->d * dv.elt / 16, static_cast<uint4 *>(xs));
  return launch_status();
}

extern "C" int moe_combine_reduce(const moe_shape *shape, const float *rows, const int32_t *topk_idx,
                                  const moe_dispatch *tables, void *y, void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!rows || !topk_idx || !y || !tables_ok(tables)) return MOE_ERR_INVALID_ARG;
  if (shape->T == 0) return MOE_OK;
  begin_launches();
  return launch_combine(shape, dv, rows, topk_idx, tables, y, false, (hipStream_t)stream);
}
