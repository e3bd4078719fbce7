"""GPU parity of the fp32 kernels without a tile table at the edges of their ranges: rows per expert around one, three and
four 32-row blocks, empty experts, large experts cut into units, more units than workgroups, reductions shorter than the waves'
shares and with partial groups, partial strips; one layer per form, and the tile kernels on the same tables."""
import numpy as np
import pytest

import gpu_util as G
from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu

# 32-row blocks at a time; rows of the local experts, d, f; experts per token, ranks of which the first is local
CASES = {
    "one_row": (1, (1, 0), 8, 8),
    "short_reduction": (1, (1, 31, 32, 0), 24, 40),
    "partial_groups": (1, (33, 7, 0, 40), 136, 264),
    "many_short": (1, (3,) * 16, 264, 1544),                               # two groups in flight
    "one_expert_has_all": (1, (24, 0, 0, 0), 1032, 520),
    "skew": (1, (200, 0, 1, 0, 0, 0, 0, 0), 520, 160),                     # seven units of one expert
    "all_local_on_one": (1, (0, 512, 0, 0, 0, 0, 0, 0), 2048, 2040, 1, 8),  # 16 units, 13 workgroups per strip in GEMM-1
    "all_local": (1, (65, 33, 97, 64, 96, 63, 31, 63), 2048, 2040, 1, 8),  # turns over experts in both GEMMs
    "turns_of_many": (1, (33,) * 15 + (1,) * 17, 264, 1000, 1, 16),        # two groups in flight, 47 units on 42
    "many_experts": (1, (2,) * 30 + (70,) + (0,) * 89 + (1, 0, 35, 5), 40, 72, 1, 2),  # numbered in two parts
    "three_blocks_one_round": (3, (64, 33, 97, 96, 1, 0, 20, 3), 520, 1000),
    "three_blocks_full": (3, (64, 65, 96, 97, 33, 60, 0, 97), 520, 1000, 2, 1),
    "three_blocks_two_rounds": (3, (64, 65, 96, 97, 33, 1, 0, 20, 3, 2, 1, 128, 0, 0, 0, 26), 520, 992, 2, 1),
    "three_blocks_large_expert": (3, (230, 0, 0, 0, 0, 2, 30, 44), 600, 1000),
    "three_blocks_turns": (3, (300, 0, 0, 0, 0, 0, 0, 20), 600, 1000),     # a workgroup's second unit, after weights asked for early
}


def layer(rows, d, f, k=1, R=1, seed=None):
    import torch
    cfg = wl.MoEConfig("f32", T=sum(rows) // k, d=d, f=f, E=len(rows) * R, k=k, R=R, local_rank_begin=0, local_rank_end=1,
                       dtype=wl.F32, router="normal", seed=sum(rows))
    rng = np.random.default_rng(d)
    flat = np.repeat(np.arange(len(rows)), rows).astype(np.int32)  # (no expert has more than T rows: a token's are distinct)
    idx = np.ascontiguousarray(rng.permutation(flat.reshape(k, cfg.T).T))
    tw = rng.uniform(0.2, 1.0, size=idx.shape).astype(np.float32)
    lay = L.MoELayer(cfg)
    lay.topk_idx.copy_(torch.from_numpy(idx).reshape(-1))
    lay.topk_w.copy_(torch.from_numpy(tw).reshape(-1))
    lay.build_dispatch()
    return cfg, lay, idx, tw


@pytest.mark.parametrize("name", list(CASES))
def test_f32_small_batch(oracle, name):
    import torch
    blocks, *sizes = CASES[name]
    cfg, lay, idx, tw = layer(*sizes)
    assert B.moe_forward_small_batch(lay.shape) == blocks
    w = wl.make_workload(cfg)
    lay.load_weights(w.W_gate, w.W_up, w.W_down)
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


# hot experts: 0.67 to 0.71 of the tile kernels' time; 1.2 to 1.7 x with workgroups that each keep to one expert
@pytest.mark.parametrize("rows,d,f,R", [((200, 20) + (2,) * 6, 1024, 1024, 8), ((300,) + (3,) * 31, 512, 1024, 8),
                                        ((400,) + (2,) * 15, 512, 1024, 8)])
def test_f32_small_batch_keeps_up_under_skew(rows, d, f, R):
    import torch
    cfg, lay, _, _ = layer(rows, d, f, 1, R)
    assert B.moe_forward_small_batch(lay.shape) == 1
    print(f"fp32 skew T={cfg.T} d={d} f={f} E_loc={cfg.E_loc}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(1)
    for name, which in (("packed_gate_up", 0), ("packed_down", 1)):  # fp32 packs are the matrices themselves
        n = B.moe_packed_weight_bytes(lay.shape, which) // 4
        setattr(lay, name, torch.randn(n, generator=gen, device="cuda").mul_(d ** -0.5).view(torch.uint8))
    x = torch.randn((cfg.T, d), generator=gen, device="cuda")
    us = G.device_us(lambda: lay.forward(x)), G.device_us(lambda: lay.forward_two_launch(x))
    assert us[0] <= 1.3 * us[1], us
