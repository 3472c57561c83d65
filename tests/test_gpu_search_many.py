"""The search's path for many rows (k_score_topk, k_topk_sort, the rescan), which
calls of T * 2H * S >= 2^26 take, at the edges of its workgroups: integer
inputs, whose scores are exact in fp32, against an exact selection.
"""
import pytest
import torch

import paper_2412_09764_amd as pk

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
    (16384, 2, 16, 64, 36, BF), (16385, 2, 16, 64, 36, BF), (33000, 1, 8, 8, 8, torch.float32),
    (9000, 4, 32, 300, 20, BF),
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
