// Host-side pieces of the C ABI that touch no device: shape validation, workspace geometry, status strings.
#include <algorithm>

#include "common.h"

namespace moe355 {

int check_shape(const moe_shape *s, Derived *out) {
  if (!s) return MOE_ERR_INVALID_ARG;
  if (s->T < 0 || s->d < 1 || s->f < 1 || s->E < 1 || s->R < 1 || s->k < 1) return MOE_ERR_INVALID_ARG;
  if (s->E % s->R != 0) return MOE_ERR_INVALID_ARG;
  if (s->k > s->E || s->k > kMaxTopK) return MOE_ERR_INVALID_ARG;
  if (s->local_rank_begin < 0 || s->local_rank_end <= s->local_rank_begin || s->local_rank_end > s->R)
    return MOE_ERR_INVALID_ARG;
  if (s->d % 8 != 0 || s->f % 8 != 0) return MOE_ERR_INVALID_ARG;
  if (s->dtype != MOE_F32 && s->dtype != MOE_BF16) return MOE_ERR_UNSUPPORTED;
  if (s->E > kMaxExperts) return MOE_ERR_UNSUPPORTED;
  if ((int64_t)s->T * s->k > (int64_t)1 << 30) return MOE_ERR_UNSUPPORTED;  // pair ids and rows are int32
  Derived d;
  d.epr = s->E / s->R;
  d.E_loc = (s->local_rank_end - s->local_rank_begin) * d.epr;
  d.e_lo = s->local_rank_begin * d.epr;
  d.pairs = (int64_t)s->T * s->k;
  d.P_cap = (int64_t)s->T * (s->k < d.E_loc ? s->k : d.E_loc);
  d.bm = s->dtype == MOE_BF16 ? kBM : kFBM;
  d.max_mtiles = (int)((d.P_cap + d.bm - 1) / d.bm) + d.E_loc;
  d.elt = s->dtype == MOE_BF16 ? 2 : 4;
  d.nt1 = s->dtype == MOE_BF16 ? ceil_div(s->f, kBN / 2) : ceil_div(s->f, kFBN);
  d.nt2 = s->dtype == MOE_BF16 ? ceil_div(s->d, kBN) : ceil_div(s->d, kFBN);
  if (out) *out = d;
  return MOE_OK;
}

FwdLayout forward_layout(const moe_shape *s, const Derived &dv) {
  FwdLayout L;
  size_t off = 0;
  auto take = [&off](size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes, 256);
    return at;
  };
  const size_t rows = (size_t)(dv.P_cap > 0 ? dv.P_cap : 1);
  L.header = take(32 * sizeof(int32_t));
  L.tickets = take(16 * kTicketStride * sizeof(int32_t));
  L.work1 = take((size_t)dv.max_mtiles * dv.nt1 * 4 * sizeof(int32_t));
  L.work2 = take((size_t)dv.max_mtiles * dv.nt2 * 4 * sizeof(int32_t));
  L.row_tok = take(rows * sizeof(int32_t));
  L.row_w = take(rows * sizeof(float));
  L.row_sole = take(rows * sizeof(int32_t));
  L.tile_ready = take((size_t)dv.max_mtiles * kReadyStride * sizeof(int32_t));
  L.row_tile = take(rows * sizeof(int32_t));
  L.tile_done = take((size_t)dv.max_mtiles * sizeof(int32_t));
  L.arrived = take((size_t)ceil_div(s->d, 32) * sizeof(int32_t));
  L.h = take(rows * (size_t)h_pitch(s, dv.elt) * dv.elt);
  L.o = take(rows * (size_t)s->d * sizeof(float));
  L.total = off;
  return L;
}

}  // namespace moe355

using namespace moe355;

extern "C" size_t moe_forward_workspace_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  return forward_layout(shape, dv).total;
}

extern "C" size_t moe_workspace_bytes(const moe_shape *shape) {
  // one buffer for both calls of a step: the dispatch scratch is dead once moe_build_dispatch's kernels have run
  return std::max(moe_dispatch_workspace_bytes(shape), moe_forward_workspace_bytes(shape));
}

// Below one M tile of rows per expert one launch, whatever its time (8 of 64 experts of 2048 x 512, 100 rows, would be the faster in
// two: 58 and 49 us).  With fuller experts by the time both GEMMs take, estimated from their flops: below about 60 us (time of the forward call in
// one launch over two: 8 experts of 2048 x 512 with 300 and 1000 rows each 1.05 and 1.01) what a workgroup pays for its queues
// and the hand-over is more than the kernel boundary, beyond it one launch is 3 % slower to 17 % faster (table at
// gemm_bf16_pipeline_kernel).  Not for matrices of 4 GiB and more, whose hand-over writes back and invalidates L2s.
int moe355::tile_gemm_launches(const moe_shape *shape, int elt) {
  if (shape->dtype != MOE_BF16) return 2;
  if ((int64_t)shape->T * shape->k < (int64_t)shape->E * kBM) return 1;
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 2;
  const int64_t widest = std::max(shape->T * (int64_t)shape->d, dv.P_cap * (int64_t)h_pitch(shape, elt)) * elt;
  if (widest >= (int64_t)1 << 32) return 2;
  const double flops = 6.0 * shape->T * shape->k * dv.E_loc / shape->E * shape->d * shape->f;
  return flops >= 60e-6 * (elt == 1 ? 1.8e15 : 1.1e15) ? 1 : 2;
}

extern "C" int moe_forward_gemm_launches(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  return stream_form(shape, dv, 2) ? 2 : tile_gemm_launches(shape, 2);
}

extern "C" int moe_fp8_forward_gemm_launches(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK || shape->dtype != MOE_BF16 || shape->d % 16 != 0 || shape->f % 16 != 0) return 0;
  return stream_form(shape, dv, 1) ? 2 : tile_gemm_launches(shape, 1);
}

extern "C" int moe_forward_small_batch(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  return stream_form(shape, dv, 2) ? 1 : f32_direct_blocks(shape, dv);
}

extern "C" size_t moe_unfused_workspace_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  const size_t rows = (size_t)(dv.P_cap > 0 ? dv.P_cap : 1);
  // fused layout + gathered copy of x [P_cap, d] + fp32 scatter target [T, d]
  return forward_layout(shape, dv).total + align_up(rows * (size_t)shape->d * dv.elt, 256) +
         align_up((size_t)(shape->T > 0 ? shape->T : 1) * shape->d * sizeof(float), 256);
}

extern "C" size_t moe_packed_weight_bytes(const moe_shape *shape, int which) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  if (which != 0 && which != 1) return 0;
  if (shape->dtype == MOE_F32) {
    const size_t one = (size_t)dv.E_loc * shape->d * shape->f * sizeof(float);
    return align_up(which == 0 ? 2 * one : one, 256);
  }
  const size_t tile = (size_t)kBN * kBK * 2;
  if (which == 0) return (size_t)dv.E_loc * ceil_div(shape->f, kBN / 2) * ceil_div(shape->d, kBK) * tile;
  return (size_t)dv.E_loc * ceil_div(shape->d, kBN) * ceil_div(shape->f, kBK) * tile;
}

extern "C" const char *moe_status_string(int status) {
  switch (status) {
    case MOE_OK: return "ok";
    case MOE_ERR_INVALID_ARG: return "invalid argument";
    case MOE_ERR_UNSUPPORTED: return "unsupported dtype or extent";
    case MOE_ERR_WORKSPACE: return "workspace missing or too small";
    case MOE_ERR_HIP: return "kernel launch failed";
    default: return "unknown status";
  }
}
