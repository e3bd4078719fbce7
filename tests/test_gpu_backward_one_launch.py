"""The two backward GEMMs as one resident launch against the form with a kernel boundary (moe_fused_backward_copies keeps
it): the same bits of dx, the gate weights' gradients and the weight gradients, with inputs that change from call to call, so
that a row handed over too early, or a line of an earlier call, would show.  Loads: even, and skewed with empty experts, tiles
of every height and experts of several tiles; a hidden size that is no multiple of a tile."""
import pytest

from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu


def layer(T, d, f, E, k, R, skew, seed):
    import torch
    cfg = wl.MoEConfig("bwd", T=T, d=d, f=f, E=E, k=k, R=R, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=3)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    W = [(randn(cfg.E_loc, a, b) * a ** -0.5).bfloat16() for a, b in ((d, f), (d, f), (f, d))]
    lay = L.MoELayer(cfg)
    bits = [L.from_device_bf16_bits(w) for w in W]
    lay.load_weights(*bits)
    lay.enable_training(*bits)
    lay.route(randn(T, E) - skew * torch.log1p(torch.arange(E, device="cuda")) - 60.0 * (torch.arange(E, device="cuda") == 5))
    lay.build_dispatch()
    x = randn(T, d).bfloat16()
    lay.forward_train(x)
    return lay, x, [randn(T, d).bfloat16() for _ in range(3)]


def outs(lay):
    return [t.clone() for t in (lay.dx, lay.d_topk_w, lay.dW_gate, lay.dW_up, lay.dW_down)]


def bounded(lay, x, dy, **kw):
    B.moe_fused_backward_bounded(lay.shape, x, dy, lay.topk_idx, lay.topk_w, lay.tables, lay.packed_down_t,
                                 lay.packed_gate_up_t, lay.kept, lay.dx, lay.d_topk_w, lay.dW_gate, lay.dW_up, lay.dW_down,
                                 lay.backward_ws, **kw)


# the range of the form: rows per expert around 64 and 76, even and skewed, ragged tiles in every direction, three M tiles; and
# outside of it, by name
@pytest.mark.parametrize("launches,T,d,f,E,k,skew", [(1, 1100, 2048, 1600, 32, 2, 0.0), (1, 2100, 2048, 1600, 32, 2, 2.0),
                                                     (1, 1250, 4104, 1728, 16, 1, 0.0), (1, 2300, 4104, 1728, 16, 2, 1.0),
                                                     (1, 2200, 4104, 2112, 8, 2, 0.0), (2, 600, 3080, 4032, 8, 1, 0.0),
                                                     (2, 2300, 3080, 4032, 8, 2, 1.0)])
def test_backward_one_launch_matches_two(launches, T, d, f, E, k, skew):
    import torch
    print(f"backward in one launch T={T} d={d} f={f} E={E} k={k} skew={skew}", flush=True)
    lay, x, dys = layer(T, d, f, E, k, 1, skew, T + d)
    assert B.moe_backward_gemm_launches(lay.shape) == launches
    run = lay.backward if launches == 1 else lambda x, dy: bounded(lay, x, dy, max_polls=1 << 22)
    want = []
    for dy in dys:
        lay.backward_copies(x, dy)
        want.append(outs(lay))
    assert not torch.equal(want[0][0], want[1][0]) and torch.isfinite(want[0][0].float()).all()
    for n in range(12):
        if n % 4 == 0:
            lay.backward_ws.fill_(0xFF)  # (NaN as bf16)
        lay.dx.fill_(float("nan"))
        run(x, dys[n % 3])
        torch.cuda.synchronize()
        for got, ref in zip(outs(lay), want[n % 3]):
            assert torch.equal(got, ref), n
    assert B.moe_forward_status(lay.backward_ws) == 0


def test_backward_wait_gives_up_cleanly():
    """Every tile of the second GEMM waits for one more tile than exists and gives up after a handful of polls: all kernels exit,
    the status word reads 1, the rows of dx with a local slot are NaN and those without stay zero; what does not hang on the
    hand-over is as ever, and the next call on the same workspace is whole again."""
    import torch
    print("backward in one launch: forced give-up", flush=True)
    lay, x, dys = layer(300, 264, 192, 16, 2, 4, 0.0, 7)
    assert B.moe_backward_gemm_launches(lay.shape) == 2  # (a small layer: by name)
    lay.backward(x, dys[0])
    good = outs(lay)
    idx = lay.topk_idx.view(300, 2)
    local = (idx < 4).any(dim=1)
    assert local.any() and not local.all()
    for polls, extra, status in ((4, 1, 1), (1 << 22, 0, 0)):
        lay.backward_ws.fill_(0xFF)
        lay.dx.fill_(123.0)
        bounded(lay, x, dys[0], max_polls=polls, wait_extra=extra)
        torch.cuda.synchronize()
        assert B.moe_forward_status(lay.backward_ws) == status
        got = outs(lay)
        for g, ref in zip(got[1:], good[1:]):
            assert torch.equal(g, ref)
        if status:
            assert got[0][local].isnan().all() and (got[0][~local] == 0).all()
        else:
            assert torch.equal(got[0], good[0])
