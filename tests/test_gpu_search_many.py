"""The search's path for many rows (k_score_topk, k_topk_sort, the rescan): calls
of T * 2H * S >= 2^26, and those past the lines of the path for few rows.

A workgroup of its scoring kernel has 4 waves of 32 tokens up to 2^15 rows
(T * 2H), 8 up to 2^16 and 16 beyond.  Small sets of tokens that the oracle can
walk are repeated until the call takes this path at a wanted number of waves,
and every repeat must give the oracle's selection.  Inputs are whole numbers
times powers of two, so scores are exact in fp32 whatever their order.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_09764_amd as pk
from tests.test_gpu_parity import (SCHEDULE_S, SCORE_RANGE_CASES, TOL_F32, h64, int_tensor,
                                   normal_tensor, normwise)

pytestmark = pytest.mark.gpu

BF = torch.bfloat16


def exact_search(q, K, k):
    """Selection of integer inputs on the GPU in whole numbers: (half_idx, idx,
    score), score descending, index ascending."""
    T, H, n = q.shape
    S, d = K.shape[2], K.shape[3]
    hi = torch.empty((T, H, 2, k), dtype=torch.int64, device=q.device)
    hz = torch.empty_like(hi)
    for h in range(H):
        for p in range(2):
            z = (q[:, h, p * d:(p + 1) * d].double() @ K[h, p].double().t().contiguous()).round().long()
            key = z * S + (S - 1 - torch.arange(S, device=q.device))
            top = torch.topk(key, k, dim=-1).values
            hz[:, h, p] = torch.div(top, S, rounding_mode="floor")
            hi[:, h, p] = S - 1 - (top - hz[:, h, p] * S)
    N = S * S
    zz = (hz[:, :, 0, :, None] + hz[:, :, 1, None, :]).reshape(T, H, -1)
    ii = (hi[:, :, 0, :, None] * S + hi[:, :, 1, None, :]).reshape(T, H, -1)
    top = torch.topk(zz * N + (N - 1 - ii), k, dim=-1).values
    score = torch.div(top, N, rounding_mode="floor")
    return hi, N - 1 - (top - score * N), score


@pytest.mark.parametrize("T,H", [(1, 4096), (7, 600)])
def test_few_tokens_of_many_heads(gpu_lib, T, H):
    """Fewer tokens than a workgroup has waves for: the waves without a token
    leave the thresholds behind the run counts alone (all scores are negative,
    so a threshold of 0 would drop every record)."""
    S, d, k = 8192, 8, 8
    print(f"[few-tokens-many-heads] {T} {H}", flush=True)
    assert T * 2 * H * S >= 1 << 26
    g = torch.Generator(device="cuda").manual_seed(500 + T)
    q = torch.randint(1, 5, (T, H, 2 * d), generator=g, device="cuda", dtype=torch.int8).to(BF)
    K = torch.randint(-64, 0, (H, 2, S, d), generator=g, device="cuda", dtype=torch.int8).to(BF)
    idx, w, score, hidx = pk.mem_search(q, K, k, want_half=True)
    torch.cuda.synchronize()
    hi, want, z = exact_search(q, K, k)
    assert torch.equal(hidx.long(), hi)
    assert torch.equal(idx, want)
    assert torch.equal(score.double(), z.double())


@pytest.mark.parametrize("T,H,d,S,k,dt", [
    # few sub-keys of many rows: the last call of the path for few rows, the first past it
    (8192, 2, 16, 100, 16, BF), (8193, 2, 16, 100, 16, BF), (33000, 1, 8, 8, 8, torch.float32),
    (20480, 2, 16, 200, 9, BF), (20481, 2, 16, 200, 9, BF), (12288, 4, 8, 300, 5, BF), (12289, 4, 8, 300, 5, BF),
    (16384, 2, 16, 64, 36, BF), (16385, 2, 16, 64, 36, BF), (24577, 2, 16, 70, 17, torch.float32),
    (16385, 4, 8, 300, 20, BF), (24576, 2, 16, 130, 40, BF), (24577, 2, 16, 130, 40, BF),
    (16384, 2, 16, 100, 64, BF), (16385, 2, 16, 100, 64, BF), (24577, 2, 16, 200, 64, BF),
    # k from 37 to 56: 2^16 or 2^15 rows x parts and one token more; k = 57 stays
    (8192, 2, 16, 513, 37, BF), (8193, 2, 16, 513, 37, BF), (4096, 2, 16, 513, 41, BF),
    (4097, 2, 16, 513, 41, BF), (4100, 4, 64, 600, 56, torch.float32), (4097, 2, 16, 513, 57, BF),
    # parts of 1024 rows: on the line and past it, by rows and by d
    (4098, 2, 64, 2049, 32, BF), (4099, 2, 64, 2049, 32, BF), (2050, 2, 256, 2049, 16, BF),
    (1500, 3, 160, 4096, 32, BF),
])
def test_both_sides_of_the_lines(gpu_lib, T, H, d, S, k, dt):
    """Calls around the sizes at which the search changes its path."""
    print(f"[lines] {T} {H} {d} {S} {k} {dt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(600 + T)
    q = torch.randint(-64, 65, (T, H, 2 * d), generator=g, device="cuda", dtype=torch.int8).to(dt)
    K = torch.randint(-64, 65, (H, 2, S, d), generator=g, device="cuda", dtype=torch.int8).to(dt)
    idx, w, score, hidx = pk.mem_search(q, K, k, want_half=True)
    torch.cuda.synchronize()
    hi, want, z = exact_search(q, K, k)
    assert torch.equal(hidx.long(), hi)
    assert torch.equal(idx, want)
    assert torch.equal(score.double(), z.double())
    assert (w - torch.softmax(z.double(), -1)).abs().max().item() <= 1e-5


def check_repeated(q, K, k, waves, ref=None):
    """The T tokens of q repeated to 2^15, 2^16 or 2^17 rows (4, 8 or 16 waves)
    less a ragged end, against the oracle (or ref: half_idx, idx, score)."""
    T, H, n = q.shape
    S = K.shape[2]
    tokens = {4: 1 << 15, 8: 1 << 16, 16: 1 << 17}[waves] // (2 * H)
    tokens -= 5 if waves == 16 or S >= 2100 else 0
    rows = tokens * 2 * H
    assert rows * S >= 1 << 26 or rows > 1 << 16, "the path for few rows"
    if ref is None:
        r = oracle.search(h64(q), h64(K), k)
        ref = [torch.from_numpy(r[x]).cuda() for x in ("half_idx", "idx", "score", "w")]
    at = torch.arange(tokens, device="cuda") % T
    idx, w, score, hidx = pk.mem_search(q.cuda()[at], K.cuda(), k, want_half=True)
    torch.cuda.synchronize()
    assert torch.equal(hidx.long(), ref[0].long()[at])
    assert torch.equal(idx, ref[1][at])
    assert torch.equal(score.double(), ref[2].double()[at])
    if len(ref) > 3:
        assert normwise(h64(w), ref[3][at].cpu().numpy()) <= TOL_F32


@pytest.mark.parametrize("waves", [4, 8, 16])
@pytest.mark.parametrize("case", SCORE_RANGE_CASES, ids=[c[0] for c in SCORE_RANGE_CASES])
def test_score_ranges(gpu_lib, case, waves):
    """Group maxima past the 16-bit float range, below it and around zero."""
    name, (qa, qb), qs, (ka, kb), ks = case
    S, H, n, k, T = 2048, 2, 512, 32, 48
    print(f"[many-range] {name} {waves}", flush=True)
    q = (int_tensor((T, H, n), 21, torch.float32, qa, qb) * qs).to(BF)
    K = (int_tensor((H, 2, S, n // 2), 22, torch.float32, ka, kb) * ks).to(BF)
    check_repeated(q, K, k, waves)


@pytest.mark.parametrize("k,waves", [(32, 4), (32, 8), (32, 16), (17, 8), (1, 16)])
@pytest.mark.parametrize("S", SCHEDULE_S)
def test_schedule_boundaries(gpu_lib, S, k, waves):
    """Every first-sweep split with ragged last chunks."""
    if S < 2048 and waves == 4:
        waves = 8  # below 2048 sub-keys the calls of 4 waves have few rows
    T, H, n = 37, 2, 32
    print(f"[many-schedule] {S} {k} {waves}", flush=True)
    q = int_tensor((T, H, n), 3000 + S + k, BF, -64, 64)
    K = int_tensor((H, 2, S, n // 2), 4000 + S + k, BF, -64, 64)
    check_repeated(q, K, k, waves)


@pytest.mark.parametrize("S,k,waves,dt", [
    (300, 16, 16, BF), (512, 36, 16, BF), (2048, 32, 4, BF), (2048, 32, 8, BF), (2048, 32, 16, BF),
    (2049, 48, 4, BF), (1024, 48, 16, BF), (4096, 64, 8, BF), (2100, 24, 8, torch.float32),
])
def test_all_ties(gpu_lib, S, k, waves, dt):
    """Equal sub-keys: the k lowest indices at both levels."""
    T, H, d = 32, 2, 32
    print(f"[many-ties] {S} {k} {waves} {dt}", flush=True)
    q = normal_tensor((T, H, 2 * d), 151, dt)
    K = torch.full((H, 2, S, d), 0.0625, dtype=dt)
    tokens = {4: 1 << 15, 8: 1 << 16, 16: 1 << 17}[waves] // (2 * H)
    idx, w, score, hidx = pk.mem_search(q.cuda().repeat(tokens // T, 1, 1), K.cuda(), k, want_half=True)
    torch.cuda.synchronize()
    want = torch.arange(k, device="cuda")
    assert (hidx == want).all() and (idx == want).all()
    assert (w - 1.0 / k).abs().max().item() <= 1e-6


@pytest.mark.parametrize("S,waves", [(900, 16), (2300, 4), (2300, 8)])
@pytest.mark.parametrize("rep,k", [(7, 32), (40, 32), (300, 32), (40, 48)])
def test_repeated_subkeys(gpu_lib, S, waves, rep, k):
    """Blocks of equal sub-keys: ties at every level."""
    T, H, n = 30, 2, 64
    print(f"[many-repeated] {S} {waves} {rep} {k}", flush=True)
    q = int_tensor((T, H, n), 152, BF)
    base = int_tensor((H, 2, S // rep + 1, n // 2), 153, BF)
    K = base[:, :, torch.arange(S) // rep].contiguous()
    check_repeated(q, K, k, waves)


@pytest.mark.parametrize("S,H,n,k,waves,dt", [
    (1024, 4, 512, 32, 8, BF), (1024, 4, 512, 32, 16, BF), (100, 2, 64, 16, 16, BF), (37, 3, 32, 36, 16, BF),
    (512, 2, 16, 1, 16, BF), (256, 2, 128, 36, 16, BF), (3000, 2, 512, 32, 4, BF), (200, 2, 128, 20, 16, torch.float32),
    (4100, 1, 512, 24, 8, BF), (90, 2, 8, 3, 16, torch.float32), (8192, 2, 96, 32, 4, BF), (1, 2, 16, 1, 16, BF),
])
def test_shapes(gpu_lib, S, H, n, k, waves, dt):
    """Sizes of tables, heads and queries that the small calls no longer bring here."""
    T = 33
    print(f"[many-shapes] {S} {H} {n} {k} {waves} {dt}", flush=True)
    q, K = int_tensor((T, H, n), 11, dt), int_tensor((H, 2, S, n // 2), 12, dt)
    check_repeated(q, K, k, waves)
