"""GPU parity of the fp32 kernels without a tile table at the edges of their ranges: rows per expert around one, three and
four 32-row blocks, empty experts, reductions shorter than the waves' shares and with partial groups, partial strips; one
layer per form, and the tile kernels on the same tables."""
import numpy as np
import pytest

import gpu_util as G
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu

# rows of the local experts, d, f
CASES = {
    "one_row": ((1, 0), 8, 8),
    "short_reduction": ((1, 31, 32, 0), 24, 40),
    "partial_groups": ((33, 7, 0, 40), 136, 264),
    "many_short": ((3,) * 16, 264, 1544),                                  # two groups in flight
    "one_expert_has_all": ((24, 0, 0, 0), 1032, 520),
    "skew": ((200, 0, 1, 0, 0, 0, 0, 0), 520, 160),                        # several turns of a workgroup
    "three_blocks": ((64, 65, 96, 97, 33, 1, 0, 90), 520, 1048),
    "three_blocks_skew": ((300, 0, 0, 0, 0, 2, 130, 64), 600, 1048),
    "three_blocks_one_round": ((64, 65, 96, 97, 33, 1, 0, 20), 520, 1000),
    "three_blocks_large_expert": ((300, 0, 0, 0, 0, 2, 30, 44), 600, 1000),  # in the workgroups an even load leaves empty
}


@pytest.mark.parametrize("name", list(CASES))
def test_f32_small_batch(oracle, name):
    import torch
    rows, d, f = CASES[name]
    cfg = wl.MoEConfig("f32", T=sum(rows), d=d, f=f, E=len(rows), k=1, R=1, local_rank_begin=0, local_rank_end=1,
                       dtype=wl.F32, router="normal", seed=sum(rows))
    w = wl.make_workload(cfg)
    rng = np.random.default_rng(d)
    idx = rng.permutation(np.repeat(np.arange(len(rows)), rows)).astype(np.int32)[:, None]
    tw = rng.uniform(0.2, 1.0, size=idx.shape).astype(np.float32)
    lay = L.MoELayer(cfg)
    lay.load_weights(w.W_gate, w.W_up, w.W_down)
    lay.topk_idx.copy_(torch.from_numpy(idx).reshape(-1))
    lay.topk_w.copy_(torch.from_numpy(tw).reshape(-1))
    lay.build_dispatch()
    x = L.to_device(w.x)
    ref = oracle.forward(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, cfg.E, cfg.R, 0, 1)
    first = None
    for form, fill in (("forward", 0xFF), ("forward", 0x3C), ("forward_two_launch", 0xFF)):
        print(f"{form} {name}", flush=True)
        lay.forward_ws.fill_(fill)
        lay.y.fill_(float("nan"))
        getattr(lay, form)(x)
        torch.cuda.synchronize()
        y = lay.y_host()
        G.check_y(y, ref, cfg.dtype)
        if form == "forward":
            assert first is None or np.array_equal(first, y)
            first = y
