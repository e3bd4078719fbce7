"""Host-only checks of the C ABI: the library loads, exports every declared symbol and rejects bad arguments
before touching a device."""
import ctypes as C
import os
import re

import pytest

from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "moe355.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"MOE355_API\s+[\w\s\*]+?\b(moe_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_symbols()
    assert {"moe_route_topk", "moe_build_dispatch", "moe_fused_forward", "moe_pack_weights"} <= set(names)
    assert len(names) >= 12
    lib = B.lib()
    for n in names:
        assert hasattr(lib, n), n


def test_status_strings():
    assert B.status_string(0) == "ok"
    for code in (-1, -2, -3, -4, -99):
        assert B.status_string(code)


def good_shape(**kw):
    base = dict(T=64, d=64, f=128, E=8, k=2, R=4, local_rank_begin=0, local_rank_end=4, dtype=B.MOE_BF16)
    base.update(kw)
    return B.make_shape(**base)


@pytest.mark.parametrize("kw", [dict(E=10, R=4), dict(k=9), dict(k=0), dict(k=33, E=64), dict(T=-1), dict(d=60),
                                dict(f=100), dict(local_rank_begin=2, local_rank_end=2), dict(local_rank_end=5),
                                dict(local_rank_begin=-1), dict(R=0)])
def test_invalid_shapes_are_rejected_everywhere(kw):
    s = good_shape(**kw)
    lib = B.lib()
    fake = 4096  # never dereferenced: validation fails first
    assert lib.moe_route_topk(C.byref(s), fake, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    assert B.moe_dispatch_workspace_bytes(s) == 0 and B.moe_forward_workspace_bytes(s) == 0
    assert B.moe_packed_weight_bytes(s, 0) == 0
    assert lib.moe_pack_weights(C.byref(s), fake, fake, fake, fake, fake, None) == B.MOE_ERR_INVALID_ARG


def test_unsupported_dtype_and_extent():
    lib = B.lib()
    assert lib.moe_route_topk(C.byref(good_shape(dtype=7)), 4096, 4096, 4096, None) == B.MOE_ERR_UNSUPPORTED
    assert lib.moe_route_topk(C.byref(good_shape(E=8192, R=1, local_rank_end=1)), 4096, 4096, 4096, None) \
        == B.MOE_ERR_UNSUPPORTED


def test_forward_rejects_misaligned_rows():
    lib = B.lib()
    s = good_shape()
    tb = B.moe_dispatch(*([4096] * 9))
    need = B.moe_forward_workspace_bytes(s)
    ok = [4096, 4096, 4096, C.byref(tb), 4096, 4096, 4096]     # x, topk_idx, topk_w, tables, gate_up, down, y
    for pos in (0, 4, 5, 6):
        args = list(ok)
        args[pos] = 4096 + 8
        assert lib.moe_fused_forward(C.byref(s), *args, 4096, need, None) == B.MOE_ERR_INVALID_ARG


def test_gemm_launch_rule_follows_rows_per_expert():
    lib = B.lib()
    assert lib.moe_forward_gemm_launches(C.byref(good_shape(T=4096, E=256, k=8, R=8))) == 1   # 128 rows per expert
    assert lib.moe_forward_gemm_launches(C.byref(good_shape(T=8192, E=256, k=8, R=8))) == 2   # 256
    assert lib.moe_forward_gemm_launches(C.byref(good_shape(T=8, E=8, k=2, R=1, local_rank_end=1, dtype=B.MOE_F32))) == 2
    assert lib.moe_forward_gemm_launches(C.byref(good_shape(E=6, R=4))) == 0                 # invalid shape
    # small batches: one weight-streaming launch per GEMM instead of the resident kernel (d, f < 512: not these)
    small = dict(E=64, k=8, R=8, local_rank_begin=0, local_rank_end=1)
    assert lib.moe_forward_gemm_launches(C.byref(good_shape(T=16, d=2048, f=768, **small))) == 2
    assert lib.moe_forward_gemm_launches(C.byref(good_shape(T=16, d=504, f=768, **small))) == 1
    assert lib.moe_forward_gemm_launches(C.byref(good_shape(T=129, d=2048, f=768, **small))) == 1
    # a small layer with many rows per expert: up to 64 tokens always, beyond only where it is the faster form
    dense = dict(E=8, k=8, R=1, local_rank_begin=0, local_rank_end=1)
    for T, d, f, launches in ((64, 1536, 1536, 2), (96, 1536, 1536, 1), (128, 2048, 1280, 1), (96, 1024, 1024, 2),
                              (128, 1536, 1024, 2), (64, 2048, 2048, 1)):
        assert lib.moe_forward_gemm_launches(C.byref(good_shape(T=T, d=d, f=f, **dense))) == launches, (T, d, f)


def test_gemm_launch_rule_follows_the_time_of_fuller_experts():
    def launches(rows, El, R, d, f, k=8):
        E = El * R
        s = good_shape(T=rows * E // k, d=d, f=f, E=E, k=k, R=R, local_rank_begin=0, local_rank_end=1)
        return B.moe_forward_gemm_launches(s), B.moe_fp8_forward_gemm_launches(s)
    # from 256 rows per expert on by the flops: 66 GFLOP in bf16, 108 in FP8
    assert launches(255, 8, 8, 2048, 512) == (1, 1) and launches(256, 8, 8, 2048, 512) == (2, 2)
    assert [launches(r, 8, 8, 2048, 512) for r in (1311, 1312, 2145, 2146)] == [(2, 2), (1, 2), (1, 2), (1, 1)]
    assert launches(256, 32, 4, 2880, 2880) == (1, 1)
    # x, or h with its rows on lines of their own, of 4 GiB: two launches (262144 tokens of 8192; 524288 rows of 4096 and 4032)
    assert [launches(1 << 18, 1, 1, d, 512, k=1) for d in (8176, 8192, 16368, 16384)] == [(1, 1), (2, 1), (2, 1), (2, 2)]
    assert [launches(1 << 19, 1, 1, 512, f, k=1) for f in (4032, 4048, 4096)] == [(1, 1), (2, 1), (2, 1)]
    # below 256 rows the resident kernel has a form for such operands
    s = good_shape(T=1 << 18, d=8192, f=512, E=2048, k=1, R=64, local_rank_begin=0, local_rank_end=1)
    assert B.moe_forward_gemm_launches(s) == 1
    # FP8: weight-streaming kernels for small batches, nothing for shapes it does not take
    assert B.moe_fp8_forward_gemm_launches(good_shape(T=16, d=512, f=512)) == 2
    assert B.moe_fp8_forward_gemm_launches(good_shape(f=72)) == 0
    assert B.moe_fp8_forward_gemm_launches(good_shape(dtype=B.MOE_F32)) == 0


def test_f32_small_batch_rule():
    form = lambda T, d, f, E, k, R: B.moe_forward_small_batch(  # noqa: E731  (one rank local)
        good_shape(T=T, d=d, f=f, E=E, k=k, R=R, local_rank_begin=0, local_rank_end=1, dtype=B.MOE_F32))
    assert form(256, 512, 1024, 8, 2, 1) == 3 and form(8, 512, 1024, 8, 2, 1) == 1
    # few rows per expert on average, but tokens enough for a large expert: the tile kernels
    for T, E, k, R in ((3000, 128, 1, 4), (6000, 256, 1, 4)):
        assert form(T, 1024, 1024, E, k, R) == 0
    assert form(1536, 1024, 1024, 64, 1, 8) == 1 and form(1537, 1024, 1024, 64, 1, 8) == 0
    # strips enough for two workgroups on every CU
    assert form(256, 1024, 1536, 32, 1, 1) == 1 and form(256, 1024, 1544, 32, 1, 1) == 0
    assert form(256, 1544, 1024, 32, 1, 1) == 0  # those of GEMM-2 count as well
    assert form(32, 1024, 3072, 32, 1, 1) == 1 and form(32, 1024, 3080, 32, 1, 1) == 0
    # more than 24 rows per expert: one block where few workgroups exist, three in nearly full rounds
    assert form(384, 1024, 512, 16, 1, 4) == 1 and form(385, 1024, 512, 8, 1, 2) == 0
    assert form(124, 936, 440, 16, 4, 1) == 0  # 31 rows: many experts have more than 32
    assert form(120, 1024, 504, 8, 2, 1) == 1 and form(300, 1024, 504, 8, 2, 1) == 0 and form(144, 512, 2048, 8, 2, 1) == 3
    for T, f, blocks in ((288, 1024, 3), (296, 1024, 0)):  # two rounds: up to 36 rows
        assert form(T, 512, f, 16, 2, 1) == blocks, T
    assert form(200, 1944, 384, 16, 4, 1) == 0 and form(200, 1944, 512, 16, 4, 1) != 1  # short reduction of GEMM-2
    assert [form(T, 512, 1024, 8, 2, 1) for T in (160, 164, 244, 248, 348, 352)] == [3, 0, 0, 3, 3, 0]  # 40, 62, 87 rows
    assert form(600, 512, 1024, 8, 2, 1) == 0 and B.moe_forward_small_batch(good_shape(E=6, R=4)) == 0
    # bf16: the weight-streaming kernels
    assert B.moe_forward_small_batch(good_shape(T=16, d=512, f=512)) == 1
    assert B.moe_forward_small_batch(good_shape(T=16, d=512, f=504)) == 0


def test_backward_gemm_launch_rule():
    def launches(rows, El, R, d, f, k=8, **kw):
        E = El * R
        assert rows * E % k == 0
        return B.moe_backward_gemm_launches(good_shape(T=rows * E // k, d=d, f=f, E=E, k=k, R=R, local_rank_begin=0,
                                                       local_rank_end=1, **kw))
    # rows per expert, by the number of experts
    assert [launches(r, 16, 8, 4096, 1536) for r in (64, 75, 76, 256, 512, 599, 600)] == [2, 2, 1, 1, 1, 1, 2]
    assert [launches(r, 32, 4, 2880, 2880) for r in (63, 64, 599, 600)] == [2, 1, 1, 2]
    # an item of the second GEMM for every CU, half of them with three M tiles per expert
    assert [launches(r, 8, 1, 4096, 14336) for r in (90, 300, 511, 512)] == [2, 2, 2, 1]
    assert [launches(r, 8, 1, 8192, 2048) for r in (90, 300)] == [1, 1] and launches(90, 8, 1, 7936, 2048) == 2
    assert launches(550, 8, 4, 2048, 4096) == 2
    # launches of less than 0.1 ms; operands of 4 GiB; shapes the backward pass does not take
    assert launches(300, 8, 8, 2048, 512) == 2
    assert launches(500, 32, 4, 4096, 16704) == 1 and launches(500, 32, 4, 4096, 16832) == 2   # 64000 rows of [dg | du]
    assert launches(500, 32, 64, 2096, 1024, k=1) == 1 and launches(500, 32, 64, 2104, 1024, k=1) == 2  # 1024000 of dy
    assert launches(300, 32, 4, 4096, 2024) == 0 and launches(300, 32, 4, 4096, 2048, dtype=B.MOE_F32) == 0
    assert B.moe_backward_gemm_launches(good_shape(E=6, R=4)) == 0


def test_forward_rejects_extents_beyond_32bit_row_offsets():
    lib = B.lib()
    s = good_shape(T=1 << 20, d=8192, f=8192, k=2)
    tb = B.moe_dispatch(*([4096] * 9))
    need = B.moe_forward_workspace_bytes(s)
    assert need > 0
    assert lib.moe_fused_forward(C.byref(s), 4096, 4096, 4096, C.byref(tb), 4096, 4096, 4096, 4096, need, None) \
        == B.MOE_ERR_UNSUPPORTED


def test_null_pointers_and_small_workspace():
    lib = B.lib()
    s = good_shape()
    fake = 4096
    assert lib.moe_route_topk(None, fake, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_topk(C.byref(s), None, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    tb = B.moe_dispatch(*([fake] * 9))
    assert lib.moe_build_dispatch(C.byref(s), None, C.byref(tb), fake, 1 << 20, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_build_dispatch(C.byref(s), fake, C.byref(tb), fake, 16, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_build_dispatch(C.byref(s), fake, C.byref(tb), None, 1 << 20, None) == B.MOE_ERR_WORKSPACE
    holes = B.moe_dispatch(*([fake] * 8 + [None]))
    assert lib.moe_build_dispatch(C.byref(s), fake, C.byref(holes), fake, 1 << 20, None) == B.MOE_ERR_INVALID_ARG
    need = B.moe_forward_workspace_bytes(s)
    args = (C.byref(s), fake, fake, fake, C.byref(tb), fake, fake, fake)
    assert lib.moe_fused_forward(*args, 4096, need - 1, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_fused_forward(*args, 4096 + 8, need, None) == B.MOE_ERR_INVALID_ARG  # misaligned workspace
    assert lib.moe_fused_forward(C.byref(s), None, fake, fake, C.byref(tb), fake, fake, fake, 4096, need, None) \
        == B.MOE_ERR_INVALID_ARG
    assert lib.moe_unfused_forward(*args, 4096, need, None) == B.MOE_ERR_WORKSPACE  # needs the larger workspace
    assert lib.moe_dispatch_gather(C.byref(s), fake, C.byref(tb), None, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_combine_reduce(C.byref(s), None, fake, C.byref(tb), fake, None) == B.MOE_ERR_INVALID_ARG


def test_sizes_for_the_named_configs():
    for name, cfg in wl.CONFIGS.items():
        s = B.shape_of(cfg)
        assert B.moe_dispatch_workspace_bytes(s) >= 64 * (cfg.E + cfg.R) * 4
        elt = 2 if cfg.dtype == wl.BF16 else 4
        raw = cfg.E_loc * cfg.d * cfg.f * elt
        assert B.moe_packed_weight_bytes(s, 0) >= 2 * raw and B.moe_packed_weight_bytes(s, 1) >= raw
        assert B.moe_packed_weight_bytes(s, 0) < 2.2 * raw + (1 << 20)
        rows = cfg.T * min(cfg.k, cfg.E_loc)
        assert B.moe_forward_workspace_bytes(s) >= rows * (cfg.f * elt + cfg.d * 4)
        assert B.moe_unfused_workspace_bytes(s) > B.moe_forward_workspace_bytes(s)


def test_t_zero_is_a_noop_on_the_host():
    s = good_shape(T=0)
    lib = B.lib()
    assert lib.moe_route_topk(C.byref(s), 4096, 4096, 4096, None) == B.MOE_OK


def test_router_logits_arguments():
    lib = B.lib()
    s = good_shape()
    need = B.moe_router_workspace_bytes(s)
    assert need >= 256 and need % 256 == 0
    assert B.moe_router_workspace_bytes(good_shape(E=0)) == 0
    fake = 4096
    assert lib.moe_router_logits(C.byref(s), None, fake, fake, fake, need, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_router_logits(C.byref(s), fake, fake, None, fake, need, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_router_logits(C.byref(s), fake + 2, fake, fake, fake, need, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_router_logits(C.byref(s), fake, fake, fake, fake, need - 1, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_router_logits(C.byref(s), fake, fake, fake, None, need, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_router_logits(C.byref(good_shape(T=0)), fake, fake, fake, fake, 1 << 20, None) == B.MOE_OK
    # the partial sums of the parts of the reduction range fit: parts <= 8
    for cfg in wl.CONFIGS.values():
        sh = B.shape_of(cfg)
        assert B.moe_router_workspace_bytes(sh) <= 8 * cfg.T * cfg.E * 4 + 512


@pytest.mark.parametrize("E,d,k", [(8, 4096, 2), (32, 2880, 4), (128, 2048, 8), (256, 7168, 8), (600, 512, 8)])
def test_router_workspaces_serve_every_smaller_batch(E, d, k):
    # sized once for the largest batch; a smaller one may be cut into more parts (at most 32 of the reduction range)
    last = (0, 0)
    for T in list(range(1, 700, 9)) + list(range(700, 20000, 77)):
        s = good_shape(T=T, d=d, E=E, k=k, R=1, local_rank_begin=0, local_rank_end=1)
        size = (B.moe_router_workspace_bytes(s), B.moe_route_from_x_workspace_bytes(s))
        assert size[0] >= last[0] and size[1] >= last[1], T
        assert max(size) <= 32 * T * E * 4 + 512 and size[1] >= T * E * 4, T
        last = size


def test_fp8_entry_points_arguments():
    lib = B.lib()
    s = good_shape()
    fake = 4096
    tb = B.moe_dispatch(*([fake] * 9))
    need = B.moe_fp8_forward_workspace_bytes(s)
    assert need > B.moe_forward_workspace_bytes(s) + s.T * s.d  # room for x as codes and its scales
    for which in (0, 1):
        raw = (s.local_rank_end - s.local_rank_begin) * (s.E // s.R) * s.d * s.f * (2 if which == 0 else 1)
        assert raw <= B.moe_fp8_packed_weight_bytes(s, which) < 2.2 * raw + (1 << 20)  # one byte per weight + padding
    assert B.moe_fp8_packed_weight_bytes(s, 2) == 0
    args = (C.byref(s), fake, fake, fake, C.byref(tb), fake, fake)
    assert lib.moe_fp8_fused_forward(*args, None, fake, fake, need, None, None) == B.MOE_ERR_INVALID_ARG  # no h_scale
    assert lib.moe_fp8_fused_forward(*args, fake, fake, fake, need - 1, None, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_fp8_fused_forward(*args, fake, None, fake, need, None, None) == B.MOE_ERR_INVALID_ARG
    odd = good_shape(d=72)  # rows are not whole 16-code chunks
    big = 1 << 30
    assert lib.moe_fp8_fused_forward(C.byref(odd), fake, fake, fake, C.byref(tb), fake, fake, fake, fake, fake, big,
                                     None, None) == B.MOE_ERR_UNSUPPORTED
    assert lib.moe_fp8_pack_weights(C.byref(odd), fake, fake, fake, fake, fake, None) == B.MOE_ERR_UNSUPPORTED
    f32 = good_shape(dtype=B.MOE_F32)
    assert lib.moe_fp8_pack_weights(C.byref(f32), fake, fake, fake, fake, fake, None) == B.MOE_ERR_UNSUPPORTED
    assert lib.moe_fp8_pack_weights(C.byref(s), fake, None, fake, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_fp8_quantize_rows(4, 12, fake, fake, fake, None) == B.MOE_ERR_INVALID_ARG   # cols % 8
    assert lib.moe_fp8_quantize_rows(4, 16, fake + 4, fake, fake, None) == B.MOE_ERR_INVALID_ARG  # misaligned
    assert lib.moe_fp8_quantize_rows(-1, 16, fake, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_fp8_quantize_rows(0, 16, fake, fake, fake, None) == B.MOE_OK
    assert lib.moe_fp8_fused_forward(C.byref(good_shape(T=0)), fake, fake, fake, C.byref(tb), fake, fake, fake, fake,
                                     fake, big, None, None) == B.MOE_OK


def test_route_gate_arguments():
    lib = B.lib()
    s = good_shape()
    fake = 4096
    assert lib.moe_route_topk_gate(C.byref(s), fake, None, 2, fake, fake, None) == B.MOE_ERR_INVALID_ARG  # gate
    assert lib.moe_route_topk_gate(C.byref(s), None, None, 1, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_topk_gate(C.byref(good_shape(k=9)), fake, None, 1, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_topk_gate(C.byref(good_shape(T=0)), fake, None, 1, fake, fake, None) == B.MOE_OK


def test_training_entry_points_arguments():
    lib = B.lib()
    s = good_shape()
    fake = 4096
    tb = B.moe_dispatch(*([fake] * 9))
    kept = B.moe_train_kept_bytes(s)
    ws = B.moe_backward_workspace_bytes(s)
    El = (s.local_rank_end - s.local_rank_begin) * (s.E // s.R)
    rows = s.T * min(s.k, El)
    assert kept >= rows * (2 * s.f * 2 + s.d * 4)           # g, u in bf16 and the weighted rows in fp32
    assert ws >= rows * (3 * s.f * 2 + s.d * 4) + (2 * s.d + 3 * s.f) * rows * 2  # intermediates + transposed operands
    assert B.moe_backward_packed_weight_bytes(s, 0) >= El * s.d * s.f * 2
    assert B.moe_backward_packed_weight_bytes(s, 1) >= 2 * El * s.d * s.f * 2
    assert B.moe_backward_packed_weight_bytes(s, 2) == 0
    fwd_ws = B.moe_forward_workspace_bytes(s)
    f_args = (C.byref(s), fake, fake, fake, C.byref(tb), fake, fake, fake)
    assert lib.moe_fused_forward_train(*f_args, fake, kept - 1, fake, fwd_ws, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_fused_forward_train(*f_args, None, kept, fake, fwd_ws, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_fused_forward_train(*f_args, fake, kept, fake, fwd_ws - 1, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_fused_forward_train(C.byref(good_shape(dtype=B.MOE_F32)), fake, fake, fake, C.byref(tb), fake, fake,
                                       fake, fake, 1 << 30, fake, 1 << 30, None) == B.MOE_ERR_UNSUPPORTED
    b_args = (C.byref(s), fake, fake, fake, fake, C.byref(tb), fake, fake, fake, kept, fake, fake)
    assert lib.moe_fused_backward(*b_args, None, None, None, fake, ws - 1, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_fused_backward(*b_args, fake, None, None, fake, ws, None) == B.MOE_ERR_INVALID_ARG  # all three or none
    assert lib.moe_fused_backward(C.byref(s), fake, None, fake, fake, C.byref(tb), fake, fake, fake, kept, fake, fake,
                                  None, None, None, fake, ws, None) == B.MOE_ERR_INVALID_ARG           # no dy
    # weight gradients leave in 16-byte stores: a pointer that is only 8-byte aligned is rejected
    assert lib.moe_fused_backward(*b_args, fake, fake + 8, fake, fake, ws, None) == B.MOE_ERR_INVALID_ARG
    odd = good_shape(f=72)  # the backward needs whole 64-index reduction tiles over f
    assert lib.moe_fused_backward(C.byref(odd), fake, fake, fake, fake, C.byref(tb), fake, fake, fake, 1 << 30, fake,
                                  fake, None, None, None, fake, 1 << 30, None) == B.MOE_ERR_UNSUPPORTED
    assert lib.moe_pack_weights_backward(C.byref(odd), fake, fake, fake, fake, fake, None) == B.MOE_ERR_UNSUPPORTED
    assert lib.moe_pack_weights_backward(C.byref(s), fake, fake, None, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    # (T = 0 launches a fill for the weight gradients, or nothing without them: exercised on the GPU)


def test_backward_refuses_before_its_first_launch():
    """Weight gradients of more tiles or rows than the grids hold: refused with nothing enqueued (here a launch would fail with
    another status)."""
    lib = B.lib()
    fake, big = 4096, 1 << 62
    tb = B.moe_dispatch(*([fake] * 9))
    many_tiles = good_shape(T=1, d=80000, f=80000, E=4096, R=1, k=1, local_rank_begin=0, local_rank_end=1)
    many_rows = good_shape(T=1 << 23, d=64, f=64, E=1, R=1, k=1, local_rank_begin=0, local_rank_end=1)
    for s, names in ((many_tiles, ["moe_fused_backward"]), (many_rows, ["moe_fused_backward", "moe_fused_backward_copies"])):
        for name in names:
            call = lambda *grads: getattr(lib, name)(C.byref(s), fake, fake, fake, fake, C.byref(tb), fake, fake, fake, big,
                                                     fake, fake, *grads, fake, big, None)
            assert call(fake, fake, fake) == B.MOE_ERR_UNSUPPORTED, name


def test_bounded_backward_arguments():
    lib = B.lib()
    fake, big = 4096, 1 << 62
    tb = B.moe_dispatch(*([fake] * 9))
    call = lambda s, grad, polls, extra: lib.moe_fused_backward_bounded(  # noqa: E731
        C.byref(s), fake, fake, fake, fake, C.byref(tb), fake, fake, fake, big, fake, fake, grad, grad, grad, fake, big, None,
        polls, extra)
    assert call(good_shape(), fake, 0, 0) == B.MOE_ERR_INVALID_ARG
    assert call(good_shape(), fake, 4, -1) == B.MOE_ERR_INVALID_ARG
    assert call(good_shape(f=72), None, 4, 0) == B.MOE_ERR_UNSUPPORTED
    # an operand of 4 GiB and more, and weight gradients that would come from transposed copies: refused before any launch
    rows = dict(E=8, R=1, k=1, local_rank_begin=0, local_rank_end=1)
    assert call(good_shape(T=1 << 18, d=8192, f=64, **rows), None, 4, 0) == B.MOE_ERR_UNSUPPORTED
    assert call(good_shape(T=1 << 18, d=64, f=4096, **rows), None, 4, 0) == B.MOE_ERR_UNSUPPORTED
    assert call(good_shape(T=(1 << 18) - 1, d=8192, f=64, **rows), fake, 4, 0) == B.MOE_ERR_UNSUPPORTED


def test_route_backward_arguments():
    lib = B.lib()
    s = good_shape()
    fake = 4096
    assert lib.moe_route_backward(C.byref(s), fake, fake, None, fake, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_backward(C.byref(s), fake, fake, fake, None, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_backward(None, fake, fake, fake, fake, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_backward(C.byref(good_shape(T=0)), fake, fake, fake, fake, None) == B.MOE_OK


def test_mfma_rate_probe_arguments():
    lib = B.lib()
    fl = C.c_double(0.0)
    assert lib.moe_probe_mfma_rate(0, 10, 4096, 1 << 20, C.byref(fl), None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_probe_mfma_rate(4, 0, 4096, 1 << 20, C.byref(fl), None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_probe_mfma_rate(4, 10, None, 1 << 20, C.byref(fl), None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_probe_mfma_rate(4, 10, 4096, 4 * 512 - 1, C.byref(fl), None) == B.MOE_ERR_WORKSPACE


def test_noalloc_dispatch_rejects_bad_arguments_before_any_device_call():
    lib = B.lib()
    s = good_shape()
    tb = B.moe_dispatch(*([4096] * 9))
    assert lib.moe_build_dispatch_noalloc(None, 4096, C.byref(tb), None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_build_dispatch_noalloc(C.byref(s), None, C.byref(tb), None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_build_dispatch_noalloc(C.byref(s), 4096, None, None) == B.MOE_ERR_INVALID_ARG
    holes = B.moe_dispatch(*([4096] * 8 + [None]))
    assert lib.moe_build_dispatch_noalloc(C.byref(s), 4096, C.byref(holes), None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_build_dispatch_noalloc(C.byref(good_shape(E=10, R=4)), 4096, C.byref(tb), None) \
        == B.MOE_ERR_INVALID_ARG
    # beyond the static scratch (E + R counters per chunk): a clear error, nothing launched
    big = good_shape(E=1024, R=1, k=2, local_rank_begin=0, local_rank_end=1)
    assert lib.moe_build_dispatch_noalloc(C.byref(big), 4096, C.byref(tb), None) == B.MOE_ERR_UNSUPPORTED
    big = good_shape(E=2048, R=2, k=2, local_rank_begin=0, local_rank_end=1)
    assert lib.moe_build_dispatch_noalloc(C.byref(big), 4096, C.byref(tb), None) == B.MOE_ERR_UNSUPPORTED


def test_one_workspace_query_covers_both_calls():
    for kw in (dict(), dict(T=4096, d=7168, f=2048, E=256, k=8, R=8, local_rank_begin=4, local_rank_end=5),
               dict(T=0), dict(dtype=B.MOE_F32)):
        s = good_shape(**kw)
        assert B.moe_workspace_bytes(s) == max(B.moe_dispatch_workspace_bytes(s), B.moe_forward_workspace_bytes(s))
        assert B.moe_workspace_bytes(s) > 0
    assert B.moe_workspace_bytes(good_shape(k=0)) == 0


def test_forward_status_and_bounded_forward_reject_bad_arguments():
    lib = B.lib()
    flag = C.c_int32(7)
    assert lib.moe_forward_status(None, C.byref(flag), None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_forward_status(4096, None, None) == B.MOE_ERR_INVALID_ARG
    s = good_shape()
    tb = B.moe_dispatch(*([4096] * 9))
    args = (C.byref(s), 4096, 4096, 4096, C.byref(tb), 4096, 4096, 4096, 4096, 1 << 30, None)
    assert lib.moe_fused_forward_bounded(*args, 0, 0) == B.MOE_ERR_INVALID_ARG       # bound below 1
    assert lib.moe_fused_forward_bounded(*args, 10, -1) == B.MOE_ERR_INVALID_ARG     # negative extra count
    ev = (C.c_void_p * 5)()
    assert lib.moe_fused_forward_resident(*args, ev, -1, 0) == B.MOE_ERR_INVALID_ARG   # negative bound
    assert lib.moe_fused_forward_resident(*args, ev, 0, -1) == B.MOE_ERR_INVALID_ARG   # negative extra count
    assert lib.moe_fused_forward_resident(C.byref(s), None, *args[2:], None, 0, 0) == B.MOE_ERR_INVALID_ARG
    small_ws = args[:9] + (16, None)
    assert lib.moe_fused_forward_resident(*small_ws, None, 0, 0) == B.MOE_ERR_WORKSPACE
    f32 = good_shape(dtype=B.MOE_F32)
    assert lib.moe_fused_forward_resident(C.byref(f32), *args[1:], None, 0, 0) == B.MOE_ERR_UNSUPPORTED  # bf16 only
    args32 = (C.byref(f32),) + args[1:]
    assert lib.moe_fused_forward_bounded(*args32, 10, 0) == B.MOE_ERR_UNSUPPORTED    # resident kernel: bf16 only


def test_route_from_x_rejects_bad_arguments():
    lib = B.lib()
    s = good_shape()
    need = B.moe_route_from_x_workspace_bytes(s)
    assert need >= s.T * s.E * 4 and B.moe_route_from_x_workspace_bytes(good_shape(k=0)) == 0
    ok = (4096, 4096, None, 4096, 4096, 4096, need, None)
    assert lib.moe_route_from_x(C.byref(good_shape(E=10, R=4)), *ok) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_from_x(C.byref(s), None, *ok[1:]) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_from_x(C.byref(s), 4096, None, *ok[2:]) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_from_x(C.byref(s), 4096, 4096, None, None, 4096, 4096, need, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_route_from_x(C.byref(s), 4104, *ok[1:]) == B.MOE_ERR_INVALID_ARG            # x not 16-byte aligned
    assert lib.moe_route_from_x(C.byref(s), 4096, 4096, None, 4096, 4096, None, need, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_route_from_x(C.byref(s), 4096, 4096, None, 4096, 4096, 4096, need - 1, None) == B.MOE_ERR_WORKSPACE
    assert lib.moe_route_from_x(C.byref(good_shape(T=0)), *ok) == B.MOE_OK                      # empty layer: a no-op
