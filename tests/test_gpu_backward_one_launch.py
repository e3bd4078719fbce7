"""The two backward GEMMs as one resident launch against the form with a kernel boundary (moe_fused_backward_copies keeps
it): the same bits of dx, the gate weights' gradients and the weight gradients, with inputs that change from call to call, so
that a row handed over too early, or a line of an earlier call, would show.  Loads: even, and skewed with empty experts, tiles
of every height and experts of several tiles; a hidden size that is no multiple of a tile."""
import pytest

from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu


# the range of the form: rows per expert around 64 and 76, even and skewed, ragged tiles in every direction, three M tiles
@pytest.mark.parametrize("T,d,f,E,k,skew", [(1100, 2048, 1792, 32, 2, 0.0), (2100, 2048, 1792, 32, 2, 2.0),
                                            (1250, 4104, 1728, 16, 1, 0.0), (2300, 4104, 1728, 16, 2, 1.0),
                                            (2200, 4104, 2112, 8, 2, 0.0)])
def test_backward_one_launch_matches_two(T, d, f, E, k, skew):
    import torch
    print(f"backward in one launch T={T} d={d} f={f} E={E} k={k} skew={skew}", flush=True)
    cfg = wl.MoEConfig("bwd", T=T, d=d, f=f, E=E, k=k, R=1, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=3)
    assert B.moe_backward_gemm_launches(B.shape_of(cfg)) == 1
    gen = torch.Generator(device="cuda").manual_seed(T + d)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    W = [(randn(E, a, b) * a ** -0.5).bfloat16() for a, b in ((d, f), (d, f), (f, d))]
    lay = L.MoELayer(cfg)
    bits = [L.from_device_bf16_bits(w) for w in W]
    lay.load_weights(*bits)
    lay.enable_training(*bits)
    lay.route(randn(T, E) - skew * torch.log1p(torch.arange(E, device="cuda")) - 60.0 * (torch.arange(E, device="cuda") == 5))
    lay.build_dispatch()
    x = randn(T, d).bfloat16()
    lay.forward_train(x)
    outs = lambda: [t.clone() for t in (lay.dx, lay.d_topk_w, lay.dW_gate, lay.dW_up, lay.dW_down)]  # noqa: E731
    dys = [randn(T, d).bfloat16() for _ in range(3)]
    want = []
    for dy in dys:
        lay.backward_copies(x, dy)
        want.append(outs())
    assert not torch.equal(want[0][0], want[1][0]) and torch.isfinite(want[0][0].float()).all()
    for n in range(12):
        if n % 4 == 0:
            lay.backward_ws.fill_(0xFF)  # (NaN as bf16)
        lay.dx.fill_(float("nan"))
        lay.backward(x, dys[n % 3])
        torch.cuda.synchronize()
        for got, ref in zip(outs(), want[n % 3]):
            assert torch.equal(got, ref), n
