"""The resident kernels' hand-over of h between the XCDs (device-scope stores, rows on lines of their own): hidden sizes
whose rows are no whole number of 128-byte lines, inputs that change from call to call, so that a line of an earlier call
would show."""
import pytest

import gpu_util as G
from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu


# rows per expert: a few, some tiles of every height, several M tiles that start inside a line of the unpadded matrix (just
# below the mean from which calls that choose by shape take two launches, and a quarter of the experts with half of the rows)
@pytest.mark.parametrize("T", [40, 600, 2040])
@pytest.mark.parametrize("form,f", [("bf16", 72), ("bf16", 200), ("bf16", 1000), ("train", 192), ("fp8", 80), ("fp8", 336)])
def test_handover_follows_changing_inputs(oracle, form, f, T):
    import numpy as np
    import torch
    d, E, k = 256, 32, 4
    print(f"hand-over {form} T={T} d={d} f={f}", flush=True)
    cfg = wl.MoEConfig("handover", T=T, d=d, f=f, E=E, k=k, R=4, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=9)
    lay = L.MoELayer(cfg)
    gen = torch.Generator(device="cuda").manual_seed(T + f)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    W = [(randn(cfg.E_loc, a, b) * a ** -0.5).bfloat16() for a, b in ((d, f), (d, f), (f, d))]
    bits = [L.from_device_bf16_bits(w) for w in W]
    xs = [randn(T, d).bfloat16() for _ in range(3)]
    lay.route(randn(T, E) + 1.5 * (torch.arange(E, device="cuda") % 4 == 0))
    lay.build_dispatch()
    assert B.moe_forward_gemm_launches(lay.shape) == 1  # (train and fp8 choose by shape)
    rows = lay.tables.counts[cfg.local_rank_begin * cfg.epr:][:cfg.E_loc]
    assert T < 2000 or (rows > 2 * 256).any()
    if form == "fp8":
        h_scale = np.full(cfg.E_loc, 0.02, dtype=np.float32)
        lay.load_weights_fp8(*bits, h_scale)
        run, first = lay.forward_fp8, lay.forward_fp8  # (one form: later calls have to repeat the first ones)
    else:
        lay.load_weights(*bits)
        first, run = lay.forward_two_launch, lay.forward_one_launch
        if form == "train":
            lay.enable_training(*bits, wgrad=False)
            run = lay.forward_train
    ws = lay.fp8_ws if form == "fp8" else lay.forward_ws
    want = []
    for x in xs:
        ws.fill_(0xFF)  # (NaN as bf16 and as a code: a row read before it was handed over would show in the first calls)
        first(x)
        want.append(lay.y.clone())
    assert not torch.equal(want[0], want[1])
    if form == "fp8":
        idx, tw = lay.topk_idx.cpu().numpy().reshape(T, k), lay.topk_w.cpu().numpy().reshape(T, k)
        for x, w in zip(xs, want):
            G.check_y(w.double().cpu().numpy(),
                      oracle.forward_fp8(L.from_device_bf16_bits(x), idx, tw, *bits, h_scale, E, cfg.R, 0, 1), wl.BF16)
    for n in range(24):
        if n % 4 == 0:
            ws.fill_(0xFF)
        lay.y.fill_(float("nan"))
        run(xs[n % 3])
        torch.cuda.synchronize()
        assert torch.equal(lay.y, want[n % 3]), (form, f, T, n)
