"""GPU parity of the small-batch kernels (one-launch tables, weight-streaming GEMMs) at the edges of their ranges."""
import numpy as np
import pytest

import gpu_util as G
from paper_2605_05607_amd import binding as B
from paper_2605_05607_amd import layer as L
from paper_2605_05607_amd import workloads as wl

pytestmark = pytest.mark.gpu


def cfg_of(**kw):
    base = dict(name="t", T=32, d=512, f=512, E=16, k=4, R=4, local_rank_begin=1, local_rank_end=3, dtype=wl.BF16,
                router="normal", seed=11)
    base.update(kw)
    return wl.MoEConfig(**base)


# pairs at and around one, two and four iterations of the workgroup; k that does not divide 64; tokens that straddle
# waves; counters that just fit the LDS and that do not (the two-kernel form)
@pytest.mark.parametrize("T,E,k,R", [(1, 1, 1, 1), (9, 8, 7, 8), (128, 256, 8, 8), (205, 64, 5, 4), (341, 12, 3, 12),
                                     (146, 128, 7, 8), (512, 256, 8, 8), (513, 256, 8, 8), (585, 300, 7, 3),
                                     (128, 32, 32, 4), (40, 1900, 20, 19), (40, 2048, 8, 2), (4096, 96, 1, 96)])
def test_small_tables_bit_exact(oracle, T, E, k, R):
    print(f"small tables T={T} E={E} k={k} R={R}", flush=True)
    rng = np.random.default_rng(T * 13 + E)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    logits[::3] = np.round(logits[::3] * 2) / 2
    logits[1::4, E // 3:E // 3 + k] += 9.0  # many tokens on the same experts
    cfg = cfg_of(T=T, E=E, k=k, R=R, d=8, f=8, local_rank_begin=0, local_rank_end=R)
    lay, got = G.run_tables(cfg, logits)
    G.assert_tables_equal(got, oracle, logits, cfg)


# the same tables from chunks of whole tokens: one chunk more than the one-launch form, the last chunk short, one to eight
# pairs per thread around their edges, counters that just fit (E + R = 1024) and that do not
@pytest.mark.parametrize("T,E,k,R", [(513, 128, 8, 8), (640, 512, 7, 8), (8192, 256, 8, 8), (8193, 256, 8, 4),
                                     (16385, 64, 8, 2), (32769, 32, 8, 1), (65600, 16, 8, 1), (700, 1016, 6, 8),
                                     (700, 1017, 6, 9), (300, 64, 32, 4), (9000, 1000, 8, 8)])
def test_chunked_tables_bit_exact(oracle, T, E, k, R):
    test_small_tables_bit_exact(oracle, T, E, k, R)


EDGES = {
    "one_token": dict(T=1),
    "rows_31": dict(T=31, router="zipf"),
    "rows_32_every_expert": dict(T=32, E=4, k=4, R=1, local_rank_begin=0, local_rank_end=1),
    "rows_33": dict(T=33, E=2, k=2, R=1, local_rank_begin=0, local_rank_end=1, d=520, f=584),
    "rows_64": dict(T=64, E=3, k=2, R=3, local_rank_begin=0, local_rank_end=3, d=1032, f=512),
    "rows_65": dict(T=65, E=2, k=2, R=2, local_rank_begin=0, local_rank_end=2, d=512, f=776),
    "rows_128_two_passes": dict(T=128, E=4, k=4, R=1, local_rank_begin=0, local_rank_end=1, d=544, f=552),
    # more than one pass over an expert that is not the first: it goes first
    "large_expert_last": dict(T=100, E=5, k=1, R=1, local_rank_begin=0, local_rank_end=1, router="zipf", seed=4),
    "large_expert_of_many": dict(T=128, E=256, k=8, R=4, local_rank_begin=0, local_rank_end=1, router="zipf", d=520, f=536),
    "no_local_row": dict(T=3, E=64, k=1, R=64, local_rank_begin=5, local_rank_end=6),
    "many_experts": dict(T=100, E=512, k=6, R=1, local_rank_begin=0, local_rank_end=1),
    "groups": dict(T=24, d=512, f=2048, E=32, k=16, R=1, local_rank_begin=0, local_rank_end=1),
    # several groups and a last strip of 8 or 16 columns: the groups' sums fill the rows of o to the last element
    "groups_last_strip_8": dict(T=33, d=520, f=1512, E=8, k=2, R=1, local_rank_begin=0, local_rank_end=1),
    "groups_last_strip_16": dict(T=128, d=1008, f=1504, E=8, k=2, R=1, local_rank_begin=0, local_rank_end=1),
    "groups_last_strip_8_one_token": dict(T=1, d=1000, f=2048, E=16, k=16, R=1, local_rank_begin=0, local_rank_end=1),
}


@pytest.mark.parametrize("name", list(EDGES))
def test_small_batch_forward(oracle, name):
    import torch
    cfg = cfg_of(**EDGES[name])
    print(f"small-batch forward {name}", flush=True)
    w = wl.make_workload(cfg)
    lay = L.MoELayer(cfg)
    lay.load_weights(w.W_gate, w.W_up, w.W_down)
    x, lg = L.to_device(w.x), L.to_device(w.logits)
    idx, tw = oracle.route_topk(w.logits, cfg.k)
    ref = oracle.forward(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, cfg.E, cfg.R, cfg.local_rank_begin,
                         cfg.local_rank_end)
    first = None
    for fill in (0xFF, 0x3C):  # the workspace's contents before the call do not matter, and the result repeats
        lay.forward_ws.fill_(fill)
        lay.y.fill_(float("nan"))
        lay.step(lg, x)
        torch.cuda.synchronize()
        G.check_y(lay.y_host(), ref, cfg.dtype)
        first = lay.y.clone() if first is None else first
        assert torch.equal(lay.y, first)
        assert B.moe_forward_status(lay.forward_ws) == 0


@pytest.mark.parametrize("name", ["one_token", "rows_33", "rows_128_two_passes", "groups", "groups_last_strip_16"])
def test_small_batch_fp8_forward(oracle, name):
    import torch
    kw = dict(EDGES[name])
    kw["f"] = kw.get("f", 512) // 16 * 16
    kw["d"] = kw.get("d", 512) // 16 * 16
    cfg = cfg_of(**kw)
    print(f"small-batch fp8 forward {name}", flush=True)
    w = wl.make_workload(cfg)
    hs = wl.fp8_h_scale(cfg)
    lay = L.MoELayer(cfg)
    lay.load_weights_fp8(w.W_gate, w.W_up, w.W_down, hs)
    x, lg = L.to_device(w.x), L.to_device(w.logits)
    lay.route(lg)
    lay.build_dispatch()
    lay.y.fill_(float("nan"))
    lay.forward_fp8(x)
    torch.cuda.synchronize()
    idx, tw = oracle.route_topk(w.logits, cfg.k)
    ref = oracle.forward_fp8(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, hs, cfg.E, cfg.R, cfg.local_rank_begin,
                             cfg.local_rank_end)
    G.check_y(lay.y_host(), ref, cfg.dtype)


# A layer whose last strip of 32 columns is short shares its strips among as many work groups as the next larger one (with
# one group per strip it takes 1.2 times as long here; runs of one side differ by 2 %).
@pytest.mark.parametrize("T", [16, 64])
def test_short_last_strip_costs_no_groups(T):
    import torch
    us = []
    for d in (1000, 1024):
        cfg = cfg_of(T=T, d=d, f=1512, E=8, k=2, R=1, local_rank_begin=0, local_rank_end=1)
        gen = torch.Generator(device="cuda").manual_seed(T)
        randn = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
        lay = L.MoELayer(cfg)
        lay.load_weights(*(L.from_device_bf16_bits((randn(8, a, b) * a ** -0.5).bfloat16())
                           for a, b in ((d, 1512), (d, 1512), (1512, d))))
        lay.route(randn(T, 8))
        lay.build_dispatch()
        x = randn(T, d).bfloat16()
        us.append(G.device_us(lambda: lay.forward(x)))
        print(f"small-batch forward T={T} d={d}: {us[-1]:.1f} us", flush=True)
    assert us[0] <= 1.1 * us[1]


# several groups per strip, and no pick on a local expert: zeros, whatever the rows of o held
@pytest.mark.parametrize("T", [1, 40])
def test_groups_without_a_local_row(T):
    import torch
    cfg = cfg_of(T=T, d=520, f=8192, E=16, k=8, R=2, local_rank_begin=1, local_rank_end=2)
    print(f"groups without a local row T={T}", flush=True)
    w = wl.make_workload(cfg)
    lay = L.MoELayer(cfg)
    lay.load_weights(w.W_gate, w.W_up, w.W_down)
    lay.topk_idx.copy_(torch.arange(8, dtype=torch.int32).repeat(T).reshape(lay.topk_idx.shape))
    lay.topk_w.fill_(0.125)
    lay.build_dispatch()
    lay.forward_ws.fill_(0xFF)
    for _ in range(2):
        lay.y.fill_(float("nan"))
        lay.forward(L.to_device(w.x))
        torch.cuda.synchronize()
        assert not lay.y[:T].any()


# fp32 reductions that end inside a load group: the padding must not meet an infinity of the row (0 * inf)
@pytest.mark.parametrize("T,d,f", [(4, 264, 40), (200, 264, 264), (4, 24, 8)])
def test_f32_reduction_tail_beside_an_infinity(T, d, f):
    import torch
    cfg = cfg_of(T=T, d=d, f=f, E=2, k=2, R=1, local_rank_begin=0, local_rank_end=1, dtype=wl.F32)
    print(f"fp32 tail T={T} d={d} f={f}", flush=True)
    rng = np.random.default_rng(d)
    x, wg, wu, wd = (rng.uniform(0.1, 1.0, sh).astype(np.float32) for sh in ((T, d), (2, d, f), (2, d, f), (2, f, d)))
    finite = x.copy()
    x[0] = np.inf  # all weights are positive: every output of this token is +inf
    lay = L.MoELayer(cfg)
    lay.load_weights(wg, wu, wd)
    lg = L.to_device(np.zeros((T, 2), np.float32))
    ys = []
    for v in (x, finite):
        lay.step(lg, L.to_device(v))
        torch.cuda.synchronize()
        ys.append(lay.y_host().copy())
    assert np.all(np.isposinf(ys[0][0]))
    assert np.array_equal(ys[0][1:], ys[1][1:]) and np.all(np.isfinite(ys[1]))


# picks that name one expert several times for a token: every slot counts, as in the tile kernels (rows of one expert beyond
# two passes, equal tokens side by side at every place of a 32-row block)
@pytest.mark.parametrize("T,k,f", [(1, 4, 512), (20, 7, 520), (32, 8, 512), (40, 5, 512), (128, 4, 1032)])
def test_small_batch_repeated_picks(oracle, T, k, f):
    import torch
    cfg = cfg_of(T=T, E=12, k=k, R=1, f=f, local_rank_begin=0, local_rank_end=1)
    print(f"small-batch forward, repeated picks T={T} k={k} f={f}", flush=True)
    w = wl.make_workload(cfg)
    rng = np.random.default_rng(T)
    idx = rng.integers(0, cfg.E, size=(T, k)).astype(np.int32)
    idx[T // 4:] = idx[T // 4:, :1]  # most tokens: every slot the same expert
    idx[T // 2:] = 3                 # and half of them the same one
    tw = rng.uniform(0.1, 1.0, size=(T, k)).astype(np.float32)
    lay = L.MoELayer(cfg)
    lay.load_weights(w.W_gate, w.W_up, w.W_down)
    lay.topk_idx.copy_(torch.from_numpy(idx).reshape(lay.topk_idx.shape))
    lay.topk_w.copy_(torch.from_numpy(tw).reshape(lay.topk_w.shape))
    lay.build_dispatch()
    lay.y.fill_(float("nan"))
    lay.forward(L.to_device(w.x))
    torch.cuda.synchronize()
    ref = oracle.forward(w.x, idx, tw, w.W_gate, w.W_up, w.W_down, cfg.E, cfg.R, 0, 1)
    G.check_y(lay.y_host(), ref, cfg.dtype)
