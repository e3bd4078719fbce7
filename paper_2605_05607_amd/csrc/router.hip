// moe_router_logits: the gate network ahead of the routing (Sec. II-A: the experts of a token are "selected by
// the gate network"; reading: a bias-free linear map, one row of W_r per expert).  logits[T,E] = x[T,d] * W_r[E,d]^T
// in fp32, summed in a fixed order, so that the routing built on it is reproducible.
#include <algorithm>
#include <cmath>

#include "gemm_pingpong.h"
#include "route_pick.h"

namespace moe355 {

constexpr int kRouterThreads = 512;  // 8 waves = 2 (token blocks) x 4 (expert blocks)
constexpr int kRouterMaxSplit = 32;
constexpr int kRouterStages = 3;
// LDS bytes of one stage for a tile of BM tokens x BN experts: x slab then W_r slab
constexpr int router_stage_bytes(int BM, int BN) { return (BM + BN) * kBK * 2; }

// One workgroup owns BM tokens (64, 128, or 256) x BN experts (128 or 256) x one contiguous part of the reduction range: the
// product is skinny (a few hundred experts), so its cost is reading x once, and cutting the reduction range is
// what gives the chip enough workgroups.  What bounds it: every workgroup pulls its whole W_r part through its CU's L2
// port next to its rows of x, (BM + BN) x 128 bytes per k-step at some 60 GB/s, and the partial sums are written and read
// back; router_plan weighs the two.  Both operands have the reduction index contiguous in memory and go straight into the LDS (chunks
// permuted as in the expert GEMMs), a ring of three stages.  A part's block is written as fp32
// to partial[part][T][E]; the kernels below add the parts in the order 0, 1, 2, ... so that the logits, and the routing
// built on them, are reproducible.
template <int BM, int BN, bool FAR>
__global__ __launch_bounds__(kRouterThreads) void router_logits_bf16_kernel(const bf16_t *__restrict__ x,
                                                                            const bf16_t *__restrict__ W,
                                                                            float *__restrict__ partial, int T, int d,
                                                                            int E, int steps_per_part, int parts) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int l31 = lane & 31, khalf = lane >> 5, sw = (lane >> 1) & 7;
  constexpr int kStage = router_stage_bytes(BM, BN), kA = BM * 128;
  constexpr int MB = BM / 64;  // 32-row token blocks per wave, and KiB of x each wave requests per slab
  constexpr int NJ = BN / 128, NW = BN / 64;  // 32-expert blocks per wave; KiB of W_r each wave requests per slab
  constexpr int kLoads = MB + NW;
  // consecutive workgroups (one per XCD) take the parts of one token tile: an XCD's L2 then holds its parts of W_r only
  const int part = blockIdx.x % parts, t0 = blockIdx.x / parts * BM, e0 = blockIdx.y * BN;
  const int KT = (d + kBK - 1) / kBK;
  const int kt_begin = min(KT, part * steps_per_part), kt_end = min(KT, kt_begin + steps_per_part);
  RowRequests<false, 1, MB, FAR> xr;
  RowRequests<false, 1, NW, FAR> wr;
  xr.init(x, d);
  wr.init(W, d);
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int row = (wave * MB + i) * 8 + (lane >> 3);
    xr.set(0, i, row, min(t0 + row, T - 1), lane);  // rows past the end: the last one, not stored
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int row = (wave * NW + i) * 8 + (lane >> 3);
    wr.set(0, i, row, min(e0 + row, E - 1), lane);
  }
  const uint32_t lds = lds_address(smem);
  const bool tail = d % kBK != 0;
  auto clip = [&](int kt) {  // before the first request of slab kt
    if (tail && kt == KT - 1) {
      xr.clip(d, KT - 1);
      wr.clip(d, KT - 1);
    }
  };
  // Requests of half a slab: those of x first, then those of W_r (the second half starts with request kFirst).
  constexpr int kFirst = (kLoads + 1) / 2;
  auto ask_one = [&](int n, int stage, int kt) {
    const uint32_t l = lds + stage * kStage;
    if (n < MB) xr.request(0, n, l + (wave * MB + n) * 1024, kt);
    else wr.request(0, n - MB, l + kA + (wave * NW + n - MB) * 1024, kt);
  };
  auto ask_half = [&](int half, int stage, int kt) {
#pragma unroll
    for (int n = half == 0 ? 0 : kFirst; n < (half == 0 ? kFirst : kLoads); ++n) ask_one(n, stage, kt);
  };
  f32x16 acc[MB][NJ];
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][j][r] = 0.f;
  // A k-step is two halves of two substeps: the next half is read while one is multiplied, the requests go out one by one
  // between the matrix instructions (in one burst they keep the waves from reading and multiplying while the CU accepts
  // them), and one barrier between the halves says that slab kt has been read and slab kt + 1 is here.
  // Measured, 256 experts, d = 7168, with the pick: 4096 tokens 30.2 us with everything read first, two barriers and the
  // requests in a burst -> 26.8 us (28 k-steps of 40 KiB per workgroup), 16 384 tokens 81 -> 71 us.
  bf16x8 fa[2][MB][2], fb[2][NJ][2];
  auto read = [&](int h, int stage, int kt) {
    const unsigned char *sA = smem + stage * kStage + (wm * (BM / 2) + l31) * 128;
    const unsigned char *sB = smem + stage * kStage + kA + (wn * 32 * NJ + l31) * 128;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int slot = (((2 * h + q) * 2 + khalf) ^ sw) * 16;
#pragma unroll
      for (int j = 0; j < NJ; ++j) fb[h][j][q] = *reinterpret_cast<const bf16x8 *>(sB + j * 4096 + slot);
#pragma unroll
      for (int mi = 0; mi < MB; ++mi) fa[h][mi][q] = *reinterpret_cast<const bf16x8 *>(sA + mi * 4096 + slot);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // products of half h of slab kt; ASK: with the requests of half `half` of slab kt_ask between them
  auto multiply = [&](int h, int kt, auto ask, int half, int stage, int kt_ask) {
    if (tail && kt == KT - 1) {  // chunks past d repeat another chunk in both operands: zero those of x
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (kt * kBK + (2 * h + q) * 16 + khalf * 8 >= d) {
#pragma unroll
          for (int mi = 0; mi < MB; ++mi) fa[h][mi][q] = bf16x8{};
        }
    }
    constexpr int N = 2 * MB * NJ;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int q = m / (MB * NJ), mi = m % (MB * NJ) / NJ, j = m % NJ;
      acc[mi][j] = mfma_bf16(fa[h][mi][q], fb[h][j][q], acc[mi][j]);
      if constexpr (decltype(ask)::value) {
        const int n0 = half == 0 ? 0 : kFirst, n = half == 0 ? kFirst : kLoads - kFirst;
#pragma unroll
        for (int a = 0; a < kLoads; ++a)
          if (a < n && (a + 1) * N / (n + 1) == m) ask_one(n0 + a, stage, kt_ask);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int S = kRouterStages;
#pragma unroll
  for (int i = 0; i < S - 1; ++i)
    if (kt_begin + i < kt_end) {
      clip(kt_begin + i);
      ask_half(0, i, kt_begin + i);
      ask_half(1, i, kt_begin + i);
    }
  int stage = 0;
  // SECOND: the second half of slab kt + S - 1 is still to be requested; FIRST: the first half of the slab behind it is
  auto k_step = [&](int kt, auto second, auto first) {
    read(1, stage, kt);
    multiply(0, kt, second, 1, stage == 0 ? S - 1 : stage - 1, kt + S - 1);
    wait_lds_reads();
    if (decltype(first)::value || kt + S <= kt_end) wait_loads<(S - 2) * kLoads>(); else wait_loads<0>();
    slot_barrier();  // slab kt has been read, slab kt + 1 is here
    const int old = stage;
    stage = stage == S - 1 ? 0 : stage + 1;
    if (decltype(first)::value || kt + 1 < kt_end) read(0, stage, kt + 1);
    if (decltype(first)::value) clip(kt + S);
    multiply(1, kt, first, 0, old, kt + S);
  };
  static_assert(S == 3, "the waits count two slabs on the way");
  if (kt_begin < kt_end) {
    if (kt_begin + S - 1 <= kt_end) wait_loads<(S - 2) * kLoads>(); else wait_loads<0>();
    slot_barrier();
    read(0, 0, kt_begin);
    if (kt_begin + S - 1 < kt_end) {
      clip(kt_begin + S - 1);
      ask_half(0, S - 1, kt_begin + S - 1);
    }
    const std::true_type yes;
    const std::false_type no;
    int kt = kt_begin;
    for (; kt + S < kt_end; ++kt) k_step(kt, yes, yes);
    if (kt + S == kt_end) k_step(kt++, yes, no);
    for (; kt < kt_end; ++kt) k_step(kt, no, no);
  }
  // accumulator register r of lane l is C[8 * (r / 4) + 4 * (l / 32) + r % 4][l % 32] of its 32 x 32 block
  float *out = partial + (size_t)part * T * E;
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int t = t0 + wm * (BM / 2) + mi * 32 + 8 * (r >> 2) + 4 * khalf + (r & 3), e = e0 + (wn * NJ + j) * 32 + l31;
        if (t < T && e < E) out[(size_t)t * E + e] = acc[mi][j][r];
      }
}

// The routing straight from the partial sums: one wave per token adds the parts of its row in the order 0, 1, 2, ...
// (the logits of router_reduce_kernel, bit for bit), keeps them in registers, lane l owning experts
// [l * PER, l * PER + PER), and picks (route_pick_registers).  The logits themselves are stored only on request.
template <int PER>
__global__ __launch_bounds__(256) void router_reduce_topk_kernel(const float *__restrict__ partial, size_t n,
                                                                 int parts, float *__restrict__ logits,
                                                                 int32_t *__restrict__ topk_idx,
                                                                 float *__restrict__ topk_w, int T, int E, int k) {
  const int lane = lane_id();
  const int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (t >= T) return;  // whole wave leaves together
  const float *row = partial + (size_t)t * E;
  RowPicker<PER> pick;
  if (PER % 4 == 0 && (E & 3) == 0) {
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
      const int e0 = lane * PER + q * 4;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (e0 < E) {  // E % 4 == 0: the four are inside together
        v = *reinterpret_cast<const float4 *>(row + e0);
        for (int p = 1; p < parts; p += 8) {  // eight parts' loads in flight
          float4 a[8];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (p + u < parts) a[u] = *reinterpret_cast<const float4 *>(row + (size_t)(p + u) * n + e0);
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (p + u < parts) {
              v.x += a[u].x; v.y += a[u].y; v.z += a[u].z; v.w += a[u].w;
            }
        }
        if (logits) *reinterpret_cast<float4 *>(logits + (size_t)t * E + e0) = v;
      }
      const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int u = 0; u < 4; ++u) pick.key[q * 4 + u] = e0 < E ? ordered_key(vv[u]) : 0u;
    }
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane * PER + i;
      float v = 0.f;
      if (e < E) {
        v = row[e];
        for (int p = 1; p < parts; p += 8) {
          float a[8];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (p + u < parts) a[u] = row[(size_t)(p + u) * n + e];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (p + u < parts) v += a[u];
        }
        if (logits) logits[(size_t)t * E + e] = v;
      }
      pick.key[i] = e < E ? ordered_key(v) : 0u;
    }
  }
  route_pick_registers<PER>(pick, E, k, t, topk_idx, topk_w);
}

// logits = partial[0] + partial[1] + ... in that order.
// (`logits` may be part 0 itself: every element is read before it is written, by the thread that writes it.)
__global__ __launch_bounds__(256) void router_reduce_kernel(const float *partial, float *logits, size_t n, int parts) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    float v = partial[i];
    for (int p = 1; p < parts; p += 8) {  // eight parts' loads in flight
      float a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (p + u < parts) a[u] = partial[(size_t)(p + u) * n + i];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (p + u < parts) v += a[u];
    }
    logits[i] = v;
  }
}

// fp32 layers: one thread per logit, fp32 fused multiply-adds in ascending reduction order (reference-grade path).
__global__ __launch_bounds__(256) void router_logits_f32_kernel(const float *__restrict__ x,
                                                                const float *__restrict__ W,
                                                                float *__restrict__ logits, int T, int d, int E) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= (size_t)T * E) return;
  const int t = (int)(i / E), e = (int)(i % E);
  const float *xr = x + (size_t)t * d, *wr = W + (size_t)e * d;
  float sum = 0.f;
  for (int c = 0; c < d; ++c) sum = fmaf(xr[c], wr[c], sum);
  logits[i] = sum;
}

}  // namespace moe355

using namespace moe355;

// Tile and number of parts of the bf16 product, by estimated time: rounds of 256 workgroups, each some 3 us of start and
// then its k-steps at what a CU pulls through its L2 port (56 GB/s) or all of them together pull of x (4.3 TB/s), plus the
// partial sums written and read back (and 0.08 us each for the latency of adding them).
// (Measured on E = 256, d = 7168: 1000 tokens 64 x 256 tiles and 16 parts 16.0 us against 20.2 us for 128 x 256 and 32 parts;
// 4096 tokens 30.0 us (4 parts) against 32.7 us (8 parts); 16384 tokens 84 us with 128 x 256 against 96 us with 64 x 256;
// E = 128, d = 2880, 8000 tokens: 24.5 us with 252 workgroups, 32.2 us with 315.)
struct RouterPlan {
  int bm, bn, parts;
};
static RouterPlan router_plan(const moe_shape *s, int T) {
  const int kt = ceil_div(s->d, kBK);
  const int bn = s->E <= 128 ? 128 : 256;
  RouterPlan best{64, bn, 1};
  double t_best = 1e30;
  for (int bm = 64; bm <= (bn == 128 ? 256 : 128); bm *= 2) {
    const double tiles = (double)ceil_div(s->E, bn) * ceil_div(T, bm);
    for (int parts = 1; parts <= std::min(kRouterMaxSplit, kt); ++parts) {
      const double rounds = std::ceil(tiles * parts / 256);
      const double cus = tiles * parts > 128 ? 256 : tiles * parts;
      const double step = std::max({0.35, (bm + bn) * 128 / 56e3, cus * bm * 128 / 4.3e6});
      const double t = rounds * (3.0 + ceil_div(kt, parts) * step) + 8.0 * parts * T * s->E / 4.2e6 + 0.08 * parts;
      if (t < t_best) {
        t_best = t;
        best = {bm, bn, parts};
      }
    }
  }
  return best;
}

static RouterPlan router_plan(const moe_shape *s) { return router_plan(s, s->T > 0 ? s->T : 1); }

static size_t router_bytes(const moe_shape *s, int64_t rows) {
  return align_up((size_t)rows * s->E * sizeof(float) + 1, 256);
}

// Rows of partial sums (parts times tokens) that this and every smaller batch needs (of at most kRouterSized tokens): a
// caller sizes its buffer once for its largest batch, and a smaller one may be cut into more parts.  Within 64 tokens the
// tile counts are the same and the parts do not increase (their sums cost T times as much), so the first batch of
// each 64 bounds its parts.
constexpr int kRouterSized = 1 << 17;
static int64_t router_rows(const moe_shape *s, bool one_part_too) {
  const int T = s->T > 0 ? s->T : 1;
  const auto rows = [&](int parts, int t) { return parts > 1 || one_part_too ? (int64_t)parts * t : 0; };
  int64_t most = rows(router_plan(s).parts, T);
  for (int t0 = 0; t0 < std::min(T, kRouterSized); t0 += 64)
    most = std::max(most, rows(router_plan(s, t0 + 1).parts, std::min(t0 + 64, T)));
  return most;
}

extern "C" size_t moe_router_workspace_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  if (shape->dtype != MOE_BF16) return 256;
  return router_bytes(shape, router_rows(shape, false));
}

extern "C" size_t moe_route_from_x_workspace_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  // the partial sums of every part (one part at least: the logits need not be stored anywhere else)
  return router_bytes(shape, shape->dtype == MOE_BF16 ? router_rows(shape, true) : shape->T > 0 ? shape->T : 1);
}

// The product into `partial` (parts > 1) or straight into `direct` (one part).
static int launch_router_gemm(const moe_shape *shape, const RouterPlan &plan, const void *x, const void *W_r,
                              float *partial, float *direct, hipStream_t st) {
  const int parts = plan.parts;
  const int steps_per_part = ceil_div(ceil_div(shape->d, kBK), parts);
  const dim3 grid((unsigned)ceil_div(shape->T, plan.bm) * parts, ceil_div(shape->E, plan.bn));
  float *out = parts > 1 ? partial : direct;
  // 32-bit offsets reach 4 GiB of either operand
  const bool far = (int64_t)std::max(shape->T, shape->E) * shape->d * 2 >= (int64_t)1 << 32;
#define MOE355_ROUTER_(BM_, BN_, FAR_)                                                                                 \
  do {                                                                                                                 \
    static std::atomic<uint64_t> done{0};                                                                              \
    const int lds = kRouterStages * router_stage_bytes(BM_, BN_);                                                      \
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&router_logits_bf16_kernel<BM_, BN_, FAR_>), lds, done))      \
      return MOE_ERR_HIP;                                                                                              \
    hipLaunchKernelGGL((router_logits_bf16_kernel<BM_, BN_, FAR_>), grid, dim3(kRouterThreads), lds, st,               \
                       static_cast<const bf16_t *>(x), static_cast<const bf16_t *>(W_r), out, shape->T, shape->d,      \
                       shape->E, steps_per_part, parts);                                                               \
  } while (0)
#define MOE355_ROUTER(BM_, BN_) \
  do { if (far) MOE355_ROUTER_(BM_, BN_, true); else MOE355_ROUTER_(BM_, BN_, false); } while (0)
  if (plan.bn == 128) {
    if (plan.bm == 64) MOE355_ROUTER(64, 128); else if (plan.bm == 128) MOE355_ROUTER(128, 128);
    else MOE355_ROUTER(256, 128);
  } else {
    if (plan.bm == 64) MOE355_ROUTER(64, 256); else MOE355_ROUTER(128, 256);
  }
#undef MOE355_ROUTER
#undef MOE355_ROUTER_
  return launch_status();
}

extern "C" int moe_router_logits(const moe_shape *shape, const void *x, const void *W_r, float *logits,
                                 void *workspace, size_t workspace_bytes, void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!x || !W_r || !logits) return MOE_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(W_r)) % 16 != 0) return MOE_ERR_INVALID_ARG;
  const RouterPlan plan = shape->dtype == MOE_BF16 ? router_plan(shape) : RouterPlan{0, 0, 1};
  const int parts = plan.parts;
  if (!workspace || workspace_bytes < router_bytes(shape, parts > 1 ? (int64_t)parts * shape->T : 0)) return MOE_ERR_WORKSPACE;
  if (shape->T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  begin_launches();
  if (shape->dtype == MOE_BF16) {
    if ((rc = launch_router_gemm(shape, plan, x, W_r, static_cast<float *>(workspace), logits, st)) != MOE_OK) return rc;
    if (parts > 1) {
      const size_t n = (size_t)shape->T * shape->E;
      hipLaunchKernelGGL(router_reduce_kernel, dim3((unsigned)std::min<size_t>(2048, (n + 255) / 256)), dim3(256), 0,
                         st, static_cast<const float *>(workspace), logits, n, parts);
    }
  } else {
    const size_t n = (size_t)shape->T * shape->E;
    hipLaunchKernelGGL(router_logits_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       static_cast<const float *>(x), static_cast<const float *>(W_r), logits, shape->T, shape->d,
                       shape->E);
  }
  return launch_status();
}

// Gate network and routing in one call: the logits are summed from the partial products inside the kernel that picks,
// and reach memory only if the caller asks for them.
extern "C" int moe_route_from_x(const moe_shape *shape, const void *x, const void *W_r, float *logits,
                                int32_t *topk_idx, float *topk_w, void *workspace, size_t workspace_bytes,
                                void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!x || !W_r || !topk_idx || !topk_w) return MOE_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(W_r)) % 16 != 0) return MOE_ERR_INVALID_ARG;
  const RouterPlan plan = shape->dtype == MOE_BF16 ? router_plan(shape) : RouterPlan{0, 0, 1};
  const int parts = plan.parts;
  if (!workspace || workspace_bytes < router_bytes(shape, (int64_t)parts * std::max(shape->T, 1))) return MOE_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % 16 != 0) return MOE_ERR_INVALID_ARG;
  if (shape->T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  begin_launches();
  float *partial = static_cast<float *>(workspace);
  const size_t n = (size_t)shape->T * shape->E;
  if (shape->dtype == MOE_BF16) {
    if ((rc = launch_router_gemm(shape, plan, x, W_r, partial, partial, st)) != MOE_OK) return rc;
  } else {
    hipLaunchKernelGGL(router_logits_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       static_cast<const float *>(x), static_cast<const float *>(W_r), partial, shape->T, shape->d,
                       shape->E);
    if ((rc = launch_status()) != MOE_OK) return rc;
  }
  if (shape->E <= 512) {
    const dim3 grid(ceil_div(shape->T, 4)), block(256);
#define MOE355_ROUTE_X(PER_)                                                                                          \
  hipLaunchKernelGGL(router_reduce_topk_kernel<PER_>, grid, block, 0, st, partial, n, parts, logits, topk_idx, topk_w, \
                     shape->T, shape->E, shape->k)
    if (shape->E <= 64) MOE355_ROUTE_X(1);
    else if (shape->E <= 128) MOE355_ROUTE_X(2);
    else if (shape->E <= 256) MOE355_ROUTE_X(4);
    else MOE355_ROUTE_X(8);
#undef MOE355_ROUTE_X
    return launch_status();
  }
  // more experts than a wave keeps in registers: add the parts in place (part 0 becomes the logits), then the routing
  // kernel that keeps its keys in the LDS
  if (parts > 1) {
    hipLaunchKernelGGL(router_reduce_kernel, dim3((unsigned)std::min<size_t>(2048, (n + 255) / 256)), dim3(256), 0, st,
                       partial, partial, n, parts);
    if ((rc = launch_status()) != MOE_OK) return rc;
  }
  if (logits) {
    if (hipMemcpyAsync(logits, partial, n * sizeof(float), hipMemcpyDeviceToDevice, st) != hipSuccess) {
      (void)hipGetLastError();
      return MOE_ERR_HIP;
    }
  }
  return moe_route_topk(shape, partial, topk_idx, topk_w, stream);
}
