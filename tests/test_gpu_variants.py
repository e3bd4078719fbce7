"""GPU parity of the kernel variants that only larger calls select: fp32 GEMM tiles, gate-network tiles, long rows of the
activation quantiser."""
import numpy as np
import pytest

import gpu_util as G
from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu

# rows of the experts' last 64-row tiles: 1, 31 to 33, 63 to 65 and 64; 116 tiles expected
F32_ROWS = (833, 863, 864, 865, 895, 896, 897, 800)


def f32_layer(d, f, seed):
    import torch
    cfg = wl.MoEConfig("f32", T=sum(F32_ROWS), d=d, f=f, E=len(F32_ROWS), k=1, R=1, local_rank_begin=0, local_rank_end=1,
                       dtype=wl.F32, router="normal", seed=seed)
    rng = np.random.default_rng(seed)
    idx = rng.permutation(np.repeat(np.arange(cfg.E), F32_ROWS)).astype(np.int32)[:, None]
    tw = rng.uniform(0.2, 1.0, size=idx.shape).astype(np.float32)
    lay = L.MoELayer(cfg)
    lay.topk_idx.copy_(torch.from_numpy(idx).reshape(-1))
    lay.topk_w.copy_(torch.from_numpy(tw).reshape(-1))
    lay.build_dispatch()
    return cfg, idx, tw, lay


# expected items of 64 x 64: 116 x 9 and 116 x 16 (both GEMMs whole items), 116 x 9 and 116 x 3 (GEMM-2 halves)
@pytest.mark.parametrize("d,f", [(1000, 520), (136, 520)])
def test_f32_forward_larger_tiles(oracle, d, f):
    import torch
    cfg, idx, tw, lay = f32_layer(d, f, d)
    print(f"fp32 forward T={cfg.T} d={d} f={f}", flush=True)
    w = wl.make_workload(cfg)
    lay.load_weights(w.W_gate, w.W_up, w.W_down)
    lay.y.fill_(float("nan"))
    lay.forward(L.to_device(w.x))
    torch.cuda.synchronize()
    ref = oracle.forward(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, cfg.E, cfg.R, 0, 1)
    G.check_y(lay.y_host(), ref, cfg.dtype)


@pytest.mark.parametrize("d,f", [(1000, 520), (136, 520)])
def test_f32_larger_tiles_beside_an_infinity(d, f):
    # the padding of the last load group must not meet an infinity of the row (0 * inf), nor reach another row
    import torch
    cfg, idx, tw, lay = f32_layer(d, f, d + 1)
    print(f"fp32 infinity T={cfg.T} d={d} f={f}", flush=True)
    rng = np.random.default_rng(d)
    x, wg, wu, wd = (rng.uniform(0.1, 1.0, sh).astype(np.float32)
                     for sh in ((cfg.T, d), (cfg.E, d, f), (cfg.E, d, f), (cfg.E, f, d)))
    rows = [0, cfg.T // 2, cfg.T - 1]
    finite = x.copy()
    x[rows] = np.inf  # all weights are positive: every output of these tokens is +inf
    lay.load_weights(wg, wu, wd)
    ys = []
    for v in (x, finite):
        lay.forward(L.to_device(v))
        torch.cuda.synchronize()
        ys.append(lay.y_host().copy())
    assert np.all(np.isposinf(ys[0][rows]))
    rest = np.delete(np.arange(cfg.T), rows)
    assert np.array_equal(ys[0][rest], ys[1][rest]) and np.all(np.isfinite(ys[1]))


# tiles of 128 x 256, 256 x 128 (two shapes each) and 128 x 128 tokens x experts; ragged tokens and experts, partial k-steps
@pytest.mark.parametrize("T,E,d", [(5003, 250, 7176), (16385, 200, 520), (5003, 7, 4104), (9001, 100, 2888), (10833, 120, 2888)])
def test_router_larger_tiles(T, E, d):
    import torch
    print(f"router T={T} E={E} d={d}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, d), generator=gen, device="cuda").bfloat16()
    W = (torch.randn((E, d), generator=gen, device="cuda") * d ** -0.5).bfloat16()
    s = B.make_shape(T, d, 8, E, 2, 1, 0, 1, B.MOE_BF16)
    out = torch.full((T, E), float("nan"), device="cuda")
    B.moe_router_logits(s, x, W, out, torch.empty(B.moe_router_workspace_bytes(s), dtype=torch.uint8, device="cuda"))
    idx = torch.full((T, 2), -1, dtype=torch.int32, device="cuda")
    wts, logits = torch.empty((T, 2), device="cuda"), torch.full((T, E), float("nan"), device="cuda")
    ws = torch.empty(B.moe_route_from_x_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    B.moe_route_from_x(s, x, W, logits, idx, wts, ws)
    torch.cuda.synchronize()
    # exact products of bf16, fp32 sums of d of them around 1: about sqrt(d) * 2^-24 (5e-6) as a root mean square
    ref = x.double() @ W.double().T
    assert (out - ref).abs().max().item() <= 1e-4
    assert torch.equal(logits, out)  # the same partial products, added in the same order
    top = out.topk(2, dim=1).values
    assert torch.equal(torch.gather(out, 1, idx.long()), top)


@pytest.mark.parametrize("rows,cols", [(5, 8200), (3, 16392)])
def test_fp8_quantize_long_rows_bit_exact(oracle, rows, cols):
    # beyond 8192 columns the rest of a row is read a second time
    import torch
    print(f"fp8 quantize rows {rows} x {cols}", flush=True)
    rng = np.random.default_rng(cols)
    a = rng.standard_normal((rows, cols)) * 10.0 ** rng.uniform(-3, 2, size=(rows, 1))
    a[0, cols - 1] = 2 * np.abs(a[0]).max()  # the largest magnitude lies in the rest
    bits = wl.f32_to_bf16_bits(a.astype(np.float32))
    codes = torch.full((rows, cols), 0xAA, dtype=torch.uint8, device="cuda")
    scales = torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
    B.moe_fp8_quantize_rows(rows, cols, L.to_device(bits), codes, scales)
    torch.cuda.synchronize()
    want_codes, want_scales = oracle.fp8_quantize(wl.bf16_bits_to_f32(bits), axis=-1)
    assert np.array_equal(scales.cpu().numpy(), want_scales)
    got = codes.cpu().numpy()
    same = (got == want_codes) | (((got | want_codes) & 0x7F) == 0)  # -0 and +0 are the same value
    assert same.all(), f"{(~same).sum()} codes differ"
