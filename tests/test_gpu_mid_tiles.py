"""GPU parity of tiles of 65 to 128 rows (the ring with one barrier per k-step) at the edges of its range: row counts at
both ends and around 32-row blocks, one to five k-steps, partial last k-steps."""
import numpy as np
import pytest

import gpu_util as G
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu

ROWS = (65, 96, 97, 128)  # of the four experts


def layer_with_rows(d, f, seed):
    import torch
    cfg = wl.MoEConfig("mid", T=sum(ROWS), d=d, f=f, E=len(ROWS), k=1, R=1, local_rank_begin=0, local_rank_end=1,
                       dtype=wl.BF16, router="normal", seed=seed)
    w = wl.make_workload(cfg)
    idx = np.random.default_rng(seed).permutation(np.repeat(np.arange(len(ROWS)), ROWS)).astype(np.int32)[:, None]
    tw = np.random.default_rng(seed + 1).uniform(0.2, 1.0, size=idx.shape).astype(np.float32)
    lay = L.MoELayer(cfg)
    lay.topk_idx.copy_(torch.from_numpy(idx).reshape(-1))
    lay.topk_w.copy_(torch.from_numpy(tw).reshape(-1))
    lay.build_dispatch()
    return cfg, w, idx, tw, lay


@pytest.mark.parametrize("d,f", [(64, 8), (72, 128), (128, 136), (192, 200), (264, 320)])
def test_mid_tiles_forward(oracle, d, f):
    import torch
    cfg, w, idx, tw, lay = layer_with_rows(d, f, d)
    lay.load_weights(w.W_gate, w.W_up, w.W_down)
    x = L.to_device(w.x)
    ref = oracle.forward(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, cfg.E, cfg.R, 0, 1)
    for form in ("forward_two_launch", "forward_one_launch", "forward_resident"):
        print(f"{form} d={d} f={f}", flush=True)
        lay.y.fill_(float("nan"))
        getattr(lay, form)(x)
        torch.cuda.synchronize()
        G.check_y(lay.y_host(), ref, cfg.dtype)


@pytest.mark.parametrize("d,f", [(64, 16), (144, 128), (272, 400)])
def test_mid_tiles_fp8_forward(oracle, d, f):
    import torch
    cfg, w, idx, tw, lay = layer_with_rows(d, f, d)
    hs = wl.fp8_h_scale(cfg)
    lay.load_weights_fp8(w.W_gate, w.W_up, w.W_down, hs)
    print(f"fp8 forward d={d} f={f}", flush=True)
    lay.y.fill_(float("nan"))
    lay.forward_fp8(L.to_device(w.x))
    torch.cuda.synchronize()
    ref = oracle.forward_fp8(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, hs, cfg.E, cfg.R, 0, 1)
    G.check_y(lay.y_host(), ref, cfg.dtype)
