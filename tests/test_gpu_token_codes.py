"""The FP8 codes made by the launch that builds the tile table, for the tokens that have a local slot: token counts around a
workgroup's waves, a batch without any local row, picks that are no expert, rows longer than a thread keeps in registers, every
expert local, and a layer whose tables take too much LDS for the form (1024 local experts)."""
import numpy as np
import pytest

import gpu_util as G
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,R,d,f", [(1, 16, 1, 4, 272, 128), (5, 16, 2, 4, 272, 128), (1000, 64, 8, 8, 272, 128),
                                         (600, 8, 2, 1, 272, 128), (70, 8, 2, 4, 8208, 64), (300, 4096, 2, 4, 32, 64)])
def test_fp8_forward_reads_codes_of_local_tokens_only(oracle, T, E, k, R, d, f):
    import torch
    print(f"token codes T={T} E={E} k={k} R={R} d={d}", flush=True)
    cfg = wl.MoEConfig("codes", T=T, d=d, f=f, E=E, k=k, R=R, local_rank_begin=0, local_rank_end=1, dtype=wl.BF16,
                       router="normal", seed=T + E)
    lay, w = L.MoELayer(cfg), wl.make_workload(cfg)
    h_scale = wl.fp8_h_scale(cfg)
    lay.load_weights_fp8(w.W_gate, w.W_up, w.W_down, h_scale)
    x = L.to_device(w.x)
    idx, tw = oracle.route_topk(w.logits, k)
    lay.topk_w.copy_(torch.from_numpy(np.ascontiguousarray(tw, dtype=np.float32).reshape(-1)).cuda())
    outside = idx.copy()
    outside[1::3] = -1
    outside[2::3, 0] = E + 7
    for picks in (idx, outside, np.full_like(idx, E - 1)):
        away = ~((picks >= 0) & (picks < E // R)).any(1)
        lay.topk_idx.copy_(torch.from_numpy(picks.reshape(-1)).cuda())
        lay.build_dispatch()
        ys = []
        for fill in (0xFF, 0x5A):
            lay.fp8_ws.fill_(fill)
            lay.y.fill_(float("nan"))
            lay.forward_fp8(x)
            torch.cuda.synchronize()
            ys.append(lay.y.clone())
        assert torch.equal(*ys)
        y = lay.y_host().reshape(T, d)
        assert np.isfinite(y).all() and (y[away] == 0).all()
        if picks is idx:
            ref = oracle.forward_fp8(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, h_scale, E, R, 0, 1).reshape(T, d)
            G.check_y(y, ref, wl.BF16)
            whole = y
        same = (picks == idx).all(1)
        assert np.array_equal(y[same], whole[same])
