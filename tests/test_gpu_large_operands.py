"""GPU parity of calls with an operand of 4 GiB or more, where a 32-bit offset no longer reaches every row: rows on both
sides of the 4 GiB mark against plain PyTorch."""
import pytest

import gpu_util as G
from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu
GIB4 = 1 << 32


def randn(shape, std, seed):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=gen, dtype=torch.bfloat16, device="cuda").mul_(std)


def router_logits(T, d, E):
    import torch
    s = B.make_shape(T, d, 8, E, 1, 1, 0, 1, B.MOE_BF16)
    x, W = randn((T, d), 1.0, T), randn((E, d), d ** -0.5, E)
    out = torch.full((T, E), float("nan"), device="cuda")
    ws = torch.empty(B.moe_router_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    B.moe_router_logits(s, x, W, out, ws)
    torch.cuda.synchronize()
    return x, W, out


def assert_logits(x, W, out):
    # fp32 sums of d products of unit-variance logits: rounding errors of the partial sums add up to about
    # sqrt(d) * 2^-24 (4e-5 at d = 524800) as a root mean square; a row read from elsewhere is off by about 1
    ref = (x.double() @ W.double().T).float()
    assert (out - ref).abs().max().item() <= 1e-3


def test_router_weights_beyond_4_gib():
    T, d, E = 5, 524800, 4096  # rows of W_r from 4092 on start beyond 4 GiB
    print(f"router logits T={T} d={d} E={E}", flush=True)
    assert E * d * 2 >= GIB4 and 4095 * d * 2 >= GIB4
    x, W, out = router_logits(T, d, E)
    for e in (0, 2048, 4064):
        assert_logits(x, W[e:e + 32], out[:, e:e + 32])


def test_router_tokens_beyond_4_gib():
    T, d, E = 524300, 4104, 24  # d % 64 = 8: the last reduction step is partial
    print(f"router logits T={T} d={d} E={E}", flush=True)
    assert (T - 8) * d * 2 >= GIB4
    x, W, out = router_logits(T, d, E)
    for t in (0, T // 2, T - 40):
        assert_logits(x[t:t + 40], W, out[t:t + 40])


# ---- expert GEMMs: the kernels with 64-bit row addresses (an operand of 4 to 8 GiB; more is refused) ----
# (d, f): x of 4 GiB and more (GEMM-1; first backward GEMM), h of 4 GiB (GEMM-2), [dg | du] of 4 GiB (second backward GEMM)
T_FAR, E_FAR = 524300, 4


def far_layer(d, f, T_FAR=T_FAR):
    import torch
    cfg = wl.MoEConfig("far", T=T_FAR, d=d, f=f, E=E_FAR, k=1, R=1, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=5)
    lay = L.MoELayer(cfg)
    W = [randn((E_FAR, a, b), a ** -0.5, 7 + i) for i, (a, b) in enumerate(((d, f), (d, f), (f, d)))]
    bits = [L.from_device_bf16_bits(w) for w in W]
    lay.load_weights(*bits)
    x = randn((T_FAR, d), 1.0, 3)
    lay.route(randn((T_FAR, E_FAR), 1.0, 4).float())
    lay.build_dispatch()
    torch.cuda.synchronize()
    # tokens on both sides of the mark, and the tokens behind the layout's first and last rows
    rows = lay.tables.perm[:T_FAR]
    toks = torch.cat([torch.arange(8, device="cuda"), torch.arange(T_FAR - 40, T_FAR, device="cuda"), rows[:8].long(),
                      rows[-40:].long()])
    return lay, W, bits, x, toks


def reference(lay, W, x, toks, dy=None):
    """y (and dx) of the given tokens in float32; k = 1, so the gate weight is 1."""
    import torch
    y, dx = [], []
    for t, e in zip(toks.tolist(), lay.topk_idx[toks].tolist()):
        wg, wu, wd = (w[e].float() for w in W)
        xt = x[t].float().requires_grad_(dy is not None)
        h = torch.nn.functional.silu(xt @ wg) * (xt @ wu)
        y.append((h @ wd).detach())
        if dy is not None:
            dx.append(torch.autograd.grad(h @ wd, xt, dy[t].float())[0])
    host = lambda rows: torch.stack(rows).double().cpu().numpy()
    return host(y), host(dx) if dy is not None else None


def sampled(out, toks):
    return out[toks].double().cpu().numpy()


@pytest.mark.parametrize("d,f", [(4104, 64), (64, 4104)])
def test_forward_beyond_4_gib(d, f):
    import torch
    assert (T_FAR - 40) * max(d, f) * 2 >= GIB4
    lay, W, _, x, toks = far_layer(d, f)
    ref, _ = reference(lay, W, x, toks)
    for name in ("forward", "forward_one_launch", "forward_resident"):
        print(f"{name} T={T_FAR} d={d} f={f}", flush=True)
        lay.y.fill_(float("nan"))
        getattr(lay, name)(x)
        torch.cuda.synchronize()
        G.check_y(sampled(lay.y, toks), ref, wl.BF16)


@pytest.mark.parametrize("d,f", [(4104, 64), (64, 2112)])
def test_training_beyond_4_gib(d, f):
    import torch
    assert (T_FAR - 40) * max(d, 2 * f) * 2 >= GIB4
    lay, W, bits, x, toks = far_layer(d, f)
    dy = randn((T_FAR, d), 1.0, 6)
    ref_y, ref_dx = reference(lay, W, x, toks, dy)
    lay.enable_training(*bits, wgrad=False)
    lay.y.fill_(float("nan"))
    lay.dx.fill_(float("nan"))
    print(f"training forward and backward T={T_FAR} d={d} f={f}", flush=True)
    lay.forward_train(x)
    lay.backward(x, dy)
    torch.cuda.synchronize()
    G.check_y(sampled(lay.y, toks), ref_y, wl.BF16)
    # dg and du are rounded to bf16 twice on the way to dx (kept g, u and their gradients): twice the forward's mean
    got = sampled(lay.dx, toks)
    assert abs(got - ref_dx).max() <= G.BF16_MAX_REL * abs(ref_dx).max()
    assert abs(got - ref_dx).mean() <= 2 * G.BF16_MEAN_REL * abs(ref_dx).mean()


# x and dy, then [dg | du], of the last size whose weight gradients come straight from the operands (a row behind the last
# one within 4 GiB - 64 KiB), and one step of the size further: the transposed copies
@pytest.mark.parametrize("T,d,f,direct", [(525304, 4088, 64, True), (525305, 4088, 64, False), (524276, 64, 2048, True),
                                          (524280, 64, 2048, False)])
def test_weight_gradients_around_4_gib(T, d, f, direct):
    import torch
    assert (max((T + 1) * d, T * 2 * f) * 2 < GIB4 - (1 << 16)) == direct
    lay, W, bits, x, _ = far_layer(d, f, T)
    dy = randn((T, d), 1.0, 6)
    lay.enable_training(*bits)
    lay.forward_train(x)
    got = (lay.dW_gate, lay.dW_up, lay.dW_down)
    for g in got:
        g.fill_(float("nan"))
    print(f"weight gradients T={T} d={d} f={f} direct={direct}", flush=True)
    lay.backward(x, dy)
    torch.cuda.synchronize()
    for e in range(E_FAR):
        wg, wu, wd = (w[e].double() for w in W)
        ref = [torch.zeros_like(w) for w in (wg, wu, wd)]
        for toks in (lay.topk_idx == e).nonzero()[:, 0].split(1 << 14):  # k = 1: the gate weight is 1
            xt, dyt = x[toks].double(), dy[toks].double()
            g, u, dh = xt @ wg, xt @ wu, dyt @ wd.T
            sg = torch.sigmoid(g)
            ref[0] += xt.T @ (dh * u * sg * (1 + g * (1 - sg)))
            ref[1] += xt.T @ (dh * g * sg)
            ref[2] += (g * sg * u).T @ dyt
        for a, r in zip(got, ref):
            err, r = (a[e].double() - r).abs(), r.abs()
            # kept g and u, dg and du (or w h) and the result rounded to bf16: twice the forward's mean
            assert err.max() <= G.BF16_MAX_REL * r.max() and err.mean() <= 2 * G.BF16_MEAN_REL * r.mean()
