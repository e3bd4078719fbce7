"""GPU parity of calls with an operand of 4 GiB or more, where a 32-bit offset no longer reaches every row: rows on both
sides of the 4 GiB mark against plain PyTorch."""
import pytest

from paper_2605_05607_amd import binding as B

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
