"""Weight gradients against autograd in float64 at the edges of their kernels: expert sizes on both sides of 64-row blocks
and of the line between the two tile sizes, experts without rows, more rows than the table of row offsets holds, widths
that are no multiple of a tile."""
import numpy as np
import pytest

import gpu_util as G
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [((1, 64, 65, 128, 0), 136, 64), ((63, 0, 127, 2), 72, 320), ((129, 192, 193, 320, 0), 264, 192),
         ((256, 130, 0, 577), 520, 448), ((7680, 7681), 72, 64), ((15400,), 64, 128)]


@pytest.mark.parametrize("rows,d,f", CASES)
def test_weight_gradients_match_autograd(rows, d, f):
    import torch
    E, T = len(rows), sum(rows)
    print(f"weight gradients rows={rows} d={d} f={f}", flush=True)
    cfg = wl.MoEConfig("wgrad", T=T, d=d, f=f, E=E, k=1, R=1, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=3)
    gen = torch.Generator(device="cuda").manual_seed(d + f)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    W = [(randn(E, a, b) * a ** -0.5).bfloat16() for a, b in ((d, f), (d, f), (f, d))]
    bits = [L.from_device_bf16_bits(w) for w in W]
    x, dy = randn(T, d).bfloat16(), randn(T, d).bfloat16()
    idx = torch.from_numpy(np.random.default_rng(d).permutation(np.repeat(np.arange(E), rows)).astype(np.int32)).cuda()
    lay = L.MoELayer(cfg)
    lay.topk_idx.copy_(idx)
    lay.topk_w.fill_(1.0)
    lay.build_dispatch()
    lay.load_weights(*bits)
    lay.enable_training(*bits)
    got = [lay.dW_gate, lay.dW_up, lay.dW_down]
    lay.forward_train(x)
    runs = []
    for fill in (0xFF, 0x7F):
        lay.backward_ws.fill_(fill)
        for g in got:
            g.fill_(float("nan"))
        lay.backward(x, dy)
        torch.cuda.synchronize()
        runs.append([g.clone() for g in got])
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    for e in range(E):
        w = [m[e].double().requires_grad_() for m in W]
        xe, ye = x[idx == e].double(), dy[idx == e].double()
        out = (torch.nn.functional.silu(xe @ w[0]) * (xe @ w[1])) @ w[2]
        ref = torch.autograd.grad(out, w, ye)
        for g, r in zip(got, ref):
            err, r = (g[e].double() - r).abs(), r.abs()
            # kept g and u, dg and du (or w h) and the result rounded to bf16: twice the forward's mean
            assert err.max() <= G.BF16_MAX_REL * max(r.max().item(), 1e-30)
            assert err.mean() <= 2 * G.BF16_MEAN_REL * max(r.mean().item(), 1e-30)


@pytest.mark.parametrize("rows,d,f", [((129, 300, 65), 520, 320), ((1, 7681), 328, 64)])
def test_a_token_of_nans_stays_with_its_expert(rows, d, f):
    """What pads an expert's rows to whole steps is zero in both operands, whatever the first and the last token hold."""
    import torch
    E, T = len(rows), sum(rows)
    print(f"weight gradients beside NaN rows={rows} d={d} f={f}", flush=True)
    cfg = wl.MoEConfig("wgrad", T=T, d=d, f=f, E=E, k=1, R=1, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=3)
    gen = torch.Generator(device="cuda").manual_seed(d + f)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    bits = [L.from_device_bf16_bits((randn(E, a, b) * a ** -0.5).bfloat16()) for a, b in ((d, f), (d, f), (f, d))]
    x, dy = randn(T, d).bfloat16(), randn(T, d).bfloat16()
    lay = L.MoELayer(cfg)
    lay.topk_idx.copy_(torch.from_numpy(np.repeat(np.arange(E), rows).astype(np.int32)).cuda())
    lay.topk_w.fill_(1.0)
    lay.build_dispatch()
    lay.load_weights(*bits)
    lay.enable_training(*bits)
    for token in (0, T - 1):
        owner = int(lay.topk_idx[token])
        grads = []
        for value in (None, float("nan"), float("inf")):
            a, b = x.clone(), dy.clone()
            if value is not None:
                a[token], b[token] = value, value
            lay.forward_train(a)
            lay.backward(a, b)
            torch.cuda.synchronize()
            grads.append([g.clone() for g in (lay.dW_gate, lay.dW_up, lay.dW_down)])
        for other in (e for e in range(E) if e != owner):
            for g in grads[1:]:
                assert all(torch.equal(p[other], q[other]) for p, q in zip(grads[0], g)), (token, other)


@pytest.mark.parametrize("rows,d,f", CASES + [((700, 0, 65, 1, 300, 64), 1032, 576)])
def test_transposed_copies_give_the_same_bits(rows, d, f):
    """The form that operands of 4 GiB and more take, on the sizes above: every output equal to the direct form's."""
    import torch
    E, T = len(rows), sum(rows)
    print(f"weight gradients, both forms rows={rows} d={d} f={f}", flush=True)
    cfg = wl.MoEConfig("wgrad", T=T, d=d, f=f, E=E, k=1, R=1, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=3)
    gen = torch.Generator(device="cuda").manual_seed(d + f)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    bits = [L.from_device_bf16_bits((randn(E, a, b) * a ** -0.5).bfloat16()) for a, b in ((d, f), (d, f), (f, d))]
    x, dy = randn(T, d).bfloat16(), randn(T, d).bfloat16()
    lay = L.MoELayer(cfg)
    lay.topk_idx.copy_(torch.from_numpy(np.random.default_rng(f).permutation(np.repeat(np.arange(E), rows)).astype(np.int32)))
    lay.topk_w.uniform_(0.1, 1.0, generator=gen)
    lay.build_dispatch()
    lay.load_weights(*bits)
    lay.enable_training(*bits)
    lay.forward_train(x)
    out = []
    for form in (lay.backward, lay.backward_copies, lay.backward_copies):
        lay.backward_ws.fill_(0xFF)
        tensors = (lay.dx, lay.d_topk_w, lay.dW_gate, lay.dW_up, lay.dW_down)
        for t in tensors:
            t.fill_(float("nan"))
        form(x, dy)
        torch.cuda.synchronize()
        out.append([t.clone() for t in tensors])
    for other in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], other))
