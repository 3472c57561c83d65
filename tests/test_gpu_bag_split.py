"""The value bag's path for few tokens (a token's lookups split over waves) at
the edges of its slabs, waves and batches of lookups, plain and gated.

Reference: the fp64 sum of the same lookups.  fp32 sums of `bag` products err by
at most (bag + 8) * 2^-24 * sum |w v| (each addition rounds once; the waves'
partial sums add at most 8 more), bf16 outputs by one rounding (2^-8 of the
value, taken as 2^-8 of the largest) on top."""
import pytest
import torch

import paper_2412_09764_amd as pk

pytestmark = pytest.mark.gpu

CASES = [
    # (T, bag, D, dtype): one lookup batch and past it, waves with nothing to
    # do, ragged slabs, every lane-group width, the last size of the split and
    # the first past it
    (1, 128, 1024, "bf16"), (1, 9, 512, "bf16"), (3, 67, 520, "bf16"), (5, 1000, 1032, "bf16"),
    (2, 8, 4096, "bf16"), (1, 64, 2048, "f32"), (7, 33, 264, "f32"), (512, 65, 2048, "bf16"),
    (513, 65, 2048, "bf16"), (9, 512, 8, "bf16"), (9, 300, 16, "bf16"), (9, 129, 24, "bf16"),
    (9, 70, 64, "bf16"), (9, 47, 120, "bf16"), (9, 40, 256, "bf16"), (9, 40, 200, "f32"),
    (4, 64, 8, "f32"), (2048, 16, 256, "bf16"), (2049, 16, 256, "bf16"),
]


@pytest.mark.parametrize("gated", [False, True], ids=["plain", "gated"])
@pytest.mark.parametrize("T,bag,D,dt", CASES)
def test_bag_of_few_tokens(gpu_lib, T, bag, D, dt, gated):
    print(f"[bag-split] {T} {bag} {D} {dt} {gated}", flush=True)
    dtype = {"bf16": torch.bfloat16, "f32": torch.float32}[dt]
    g = torch.Generator().manual_seed(1000 + T + bag + D)
    N = 977
    V = torch.randn((N, D), generator=g).to(dtype).cuda()
    idx = torch.randint(0, N, (T, bag), generator=g).cuda()
    w = torch.randn((T, bag), generator=g).cuda()
    gate = torch.randn((T, D), generator=g).to(dtype).cuda()
    ref = torch.empty((T, D), dtype=torch.float64, device="cuda")
    mag = 0.0
    for t in range(0, T, 64):
        prod = w[t:t + 64, :, None].double() * V[idx[t:t + 64]].double()
        ref[t:t + 64] = prod.sum(1)
        mag = max(mag, prod.abs().sum(1).max().item())
    tol = (bag + 8) * 2 ** -24 * mag
    if gated:
        out, y = pk.mem_bag_forward_gated(V, idx, w, gate)
        torch.cuda.synchronize()
        s = gate.double() * torch.sigmoid(gate.double())
        # the gate's fp32 silu is within a few units of 2^-23 of its value
        want, bound = ref * s, tol * s.abs().max().item() + 8 * 2 ** -23 * (ref * s).abs().max().item()
        got = [(out, want, bound), (y, ref, tol)]
    else:
        got = [(pk.mem_bag_forward(V, idx, w), ref, tol)]
        torch.cuda.synchronize()
    for a, b, t in got:
        if dtype is torch.bfloat16:
            t = t + 2 ** -8 * b.abs().max().item()
        assert (a.double() - b).abs().max().item() <= t


@pytest.mark.parametrize("T,bag,D,dt", [(1, 9, 512, "bf16"), (3, 67, 520, "bf16"), (7, 33, 264, "f32"),
                                        (9, 70, 64, "bf16"), (9, 300, 16, "bf16"), (4, 64, 8, "f32"),
                                        (1, 128, 1024, "bf16")])
def test_infinite_weight_stays_infinite(gpu_lib, T, bag, D, dt):
    """An infinite weight on a positive row gives +inf, wherever in the bag it
    stands: no lookup past a wave's own takes part."""
    print(f"[bag-split-inf] {T} {bag} {D} {dt}", flush=True)
    dtype = {"bf16": torch.bfloat16, "f32": torch.float32}[dt]
    V = torch.ones((5, D), dtype=dtype, device="cuda")
    idx = torch.arange(bag).remainder(5).repeat(T, 1).cuda()
    for j in sorted({0, 1, 8, bag // 2, bag - 1}):
        w = torch.ones((T, bag), device="cuda")
        w[:, j] = float("inf")
        y = pk.mem_bag_forward(V, idx, w)
        torch.cuda.synchronize()
        assert (y == float("inf")).all(), j


@pytest.mark.parametrize("T,bag,D,dt", [
    (1024, 64, 64, "bf16"), (1025, 64, 64, "bf16"), (768, 32, 128, "bf16"), (769, 32, 128, "bf16"),
    (512, 16, 256, "bf16"), (513, 16, 256, "bf16"), (512, 8, 512, "bf16"), (513, 8, 512, "bf16"),
    (512, 16, 1024, "bf16"), (513, 16, 1024, "bf16"), (256, 8, 2048, "f32"), (257, 8, 2048, "f32"),
])
def test_both_sides_of_the_token_line(gpu_lib, T, bag, D, dt):
    """The last call of few tokens to a bag, and the next."""
    test_bag_of_few_tokens(gpu_lib, T, bag, D, dt, False)
