"""The search's path for few rows (sub-keys split over workgroups) at the edges
of its parts, against the oracle and against the path for many rows.

Both paths form a score by the same chain of matrix instructions and select in
the same total order, so the same queries repeated until the call takes the
path for many rows must give the same selection and, to k = 32, bitwise the
same scores; weights differ by the softmax's summation order at most (64
terms: 1e-6; with k > 32 also by the scores')."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_09764_amd as pk
from tests.test_gpu_parity import TOL_F32, h64, int_tensor, normal_tensor, normwise

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32
CASES = [
    # (S, H, n, k, T, dtype): last and single rows of a part, one part and one
    # more, every part size, T below / at / past a group of 32
    (64, 1, 64, 8, 5, F32),
    (255, 2, 64, 32, 31, BF),
    (257, 2, 48, 33, 33, BF),
    (512, 4, 512, 32, 600, BF),      # 512 keys per part, one part
    (513, 1, 160, 64, 32, BF),       # ... and one key in the second
    (700, 3, 320, 17, 300, BF),
    (1025, 2, 128, 20, 16, F32),
    (2048, 4, 512, 32, 2000, BF),    # several groups per workgroup
    (2049, 1, 512, 40, 33, BF),      # 1024 keys per part
    (4096, 1, 80, 64, 64, BF),
    (4097, 2, 512, 20, 40, BF),      # 32 slots per part, exactly the top k in each
    (8192, 2, 512, 32, 3, BF),       # 16 parts
    (8192, 1, 512, 32, 33, BF),
    (1000, 2, 24, 1, 1, F32),
]


def _ids(c):
    return f"S{c[0]}_H{c[1]}_n{c[2]}_k{c[3]}_T{c[4]}_{'f32' if c[5] is F32 else 'bf16'}"


@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_few_rows_exact(gpu_lib, case):
    S, H, n, k, T, dt = case
    print(f"[few-rows] {case}", flush=True)
    T = min(T, 100)  # the oracle walks token by token
    q, K = int_tensor((T, H, n), 211, dt), int_tensor((H, 2, S, n // 2), 212, dt)
    idx, w, score, hidx = pk.mem_search(q.cuda(), K.cuda(), k, want_half=True)
    torch.cuda.synchronize()
    ref = oracle.search(h64(q), h64(K), k)  # integers: ties at every level
    np.testing.assert_array_equal(hidx.cpu().numpy(), ref["half_idx"])
    np.testing.assert_array_equal(idx.cpu().numpy(), ref["idx"])
    np.testing.assert_array_equal(h64(score), ref["score"])
    assert normwise(h64(w), ref["w"]) <= TOL_F32


@pytest.mark.parametrize("ints", [False, True], ids=["float", "int"])
@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_few_rows_equal_many_rows(gpu_lib, case, ints):
    S, H, n, k, T, dt = case
    print(f"[few-many] {case} {ints}", flush=True)
    if ints:
        q, K = int_tensor((T, H, n), 213, dt).cuda(), int_tensor((H, 2, S, n // 2), 214, dt).cuda()
    else:
        q = normal_tensor((T, H, n), 215, dt).cuda()
        K = normal_tensor((H, 2, S, n // 2), 216, dt, 0.1).cuda()
    idx, w, score, hidx = pk.mem_search(q, K, k, want_half=True)
    reps = -(-(1 << 26) // (2 * T * H * S))  # rows * S >= 2^26
    big = q.repeat(reps, 1, 1)
    i2, w2, s2, h2 = pk.mem_search(big, K, k, want_half=True)
    torch.cuda.synchronize()
    for a, b in ((idx, i2), (hidx, h2)):
        assert torch.equal(a.expand(reps, *a.shape), b.view(reps, *a.shape))
    if k <= 32:
        assert torch.equal(score.expand(reps, *score.shape), s2.view(reps, *score.shape))
    else:
        # the path for many rows rescans rows with more than 256 candidates with
        # serial fp32 sums: each of the two differs from the exact score of n
        # products by at most n * 2^-24 * sum |q k|
        mag = (q.float().abs().amax(0).sum(-1) * K.float().abs().max()).max().item()
        assert (score - s2.view(reps, *score.shape)).abs().max().item() <= 2 * n * 2 ** -24 * mag
    assert (w - w2.view(reps, *w.shape)).abs().max().item() <= (1e-6 if k <= 32 else 1e-5)


@pytest.mark.parametrize("T", [7, 300])
def test_few_rows_variants_equal_many_rows(gpu_lib, T):
    """Query normalisation, extra pairs and the sink over the split."""
    S, H, n, k, r = 1500, 2, 320, 24, 5
    q = (normal_tensor((T, H, n), 217, BF) * 2 + 0.5).cuda()
    K = normal_tensor((H, 2, S, n // 2), 218, BF, 0.1).cuda()
    ks = normal_tensor((H, n), 219, BF, 0.1).cuda()
    g = torch.Generator().manual_seed(220)
    ex = torch.randint(0, S * S, (T, H, r), generator=g).cuda()
    reps = -(-(1 << 26) // (2 * T * H * S))
    big, exb = q.repeat(reps, 1, 1), ex.repeat(reps, 1, 1)
    print(f"[few-variants] T={T}", flush=True)
    for few, many in (
            (pk.mem_search_qnorm(q, K, k)[:3], pk.mem_search_qnorm(big, K, k)[:3]),
            (pk.mem_search_extra(q, K, k, ex)[:3], pk.mem_search_extra(big, K, k, exb)[:3]),
            (pk.mem_search_sink(q, K, k, ks, S * S, ex)[:3],
             pk.mem_search_sink(big, K, k, ks, S * S, exb)[:3]),
            (pk.mem_search_sink(q, K, k, ks, S * S)[:3],
             pk.mem_search_sink(big, K, k, ks, S * S)[:3])):
        torch.cuda.synchronize()
        idx, w, score = few
        assert torch.equal(idx.expand(reps, *idx.shape), many[0].view(reps, *idx.shape))
        assert torch.equal(score[..., :k].expand(reps, *score[..., :k].shape),
                           many[2].view(reps, *score.shape)[..., :k])
        # the sink's score is one fp32 dot of n products, summed in another order
        scale = score.abs().max().item()
        assert (score - many[2].view(reps, *score.shape)).abs().max().item() <= n * 2 ** -23 * scale
        assert (w - many[1].view(reps, *w.shape)).abs().max().item() <= 1e-5


@pytest.mark.parametrize("S,dt", [(300, F32), (512, BF), (2049, BF)])
def test_few_rows_products_past_the_float_range(gpu_lib, S, dt):
    """Finite inputs whose products overflow to -inf for all but m < k sub-keys:
    the half lists go on with the -inf rows in index order, and no rank pair
    reads an empty record."""
    H, d, k, m, T = 2, 32, 8, 5, 3
    q, K = int_tensor((T, H, 2 * d), 311, dt), int_tensor((H, 2, S, d), 312, dt)
    q[:, :, 0] = q[:, :, d] = 1e30
    K[..., 0] = -3e38
    K[:, :, [S - 1, 7, S // 2, 64, 3], 0] = 0
    assert torch.isfinite(q).all() and torch.isfinite(K).all()
    idx, w, score, hidx = pk.mem_search(q.cuda(), K.cuda(), k, want_half=True)
    torch.cuda.synchronize()
    qd = q.double().reshape(T, H, 2, d)
    z = torch.einsum("thpd,hpsd->thps", qd, K.double())
    z[z < -3.4e38] = -float("inf")
    order = torch.sort(z, dim=-1, descending=True, stable=True)
    hv, hi = order.values[..., :k], order.indices[..., :k]
    assert torch.isinf(hv[..., m:]).all() and torch.isfinite(hv[..., :m]).all()
    np.testing.assert_array_equal(hidx.cpu().numpy(), hi.numpy())
    zz = (hv[:, :, 0, :m, None] + hv[:, :, 1, None, :m]).reshape(T, H, -1)
    ii = (hi[:, :, 0, :m, None] * S + hi[:, :, 1, None, :m]).reshape(T, H, -1)
    ii, o = torch.sort(ii, dim=-1)  # equal sums: lower index first
    zz = torch.gather(zz, -1, o)
    zz, o = torch.sort(zz, dim=-1, descending=True, stable=True)
    np.testing.assert_array_equal(idx.cpu().numpy(), torch.gather(ii, -1, o)[..., :k].numpy())
    np.testing.assert_array_equal(h64(score), zz[..., :k].numpy())
    assert normwise(h64(w), torch.softmax(zz[..., :k], -1).numpy()) <= TOL_F32


def _with_nan_rows(S, H, d, T, nan, seed):
    """Integer queries and sub-keys whose products overflow with both signs for
    the sub-keys of `nan` (so that their scores are no number): all inputs
    finite.  bf16 only: in fp32 the chain's steps are fused, and +inf plus an
    unrounded product stays +inf.  Returns q, K and the exact scores with those
    at -inf."""
    q, K = int_tensor((T, H, 2 * d), seed, BF), int_tensor((H, 2, S, d), seed + 1, BF)
    for p in (0, d):
        q[:, :, p] = q[:, :, p + 16] = 1e30
    K[..., 0] = K[..., 16] = 0
    # in different steps of the product's chain: +inf first, then -inf added
    K[:, :, nan, 0], K[:, :, nan, 16] = 3e38, -3e38
    assert torch.isfinite(q).all() and torch.isfinite(K).all()
    z = torch.matmul(q.double().reshape(T, H, 2, 1, d), K.double().transpose(-1, -2).contiguous()[None])
    z = z.reshape(T, H, 2, S)
    z[..., nan] = -float("inf")
    return q, K, z


@pytest.mark.parametrize("S,k,T", [(512, 64, 40), (700, 48, 33), (300, 64, 5), (2049, 64, 33),
                                   (8192, 32, 33), (1000, 17, 33)])
def test_few_rows_scores_that_are_no_number(gpu_lib, S, k, T):
    """Sub-keys whose score is no number are never selected while k others are
    there, also where a part has more records than slots (ties, k = 64)."""
    print(f"[few-nan] {S} {k} {T}", flush=True)
    H, d = 2, 32
    nan = torch.rand(S, generator=torch.Generator().manual_seed(S)) < 0.3
    nan[S - 1] = nan[0] = True
    q, K, z = _with_nan_rows(S, H, d, T, nan, 411)
    idx, w, score, hidx = pk.mem_search(q.cuda(), K.cuda(), k, want_half=True)
    torch.cuda.synchronize()
    order = torch.sort(z, dim=-1, descending=True, stable=True)
    hv, hi = order.values[..., :k], order.indices[..., :k]
    assert torch.isfinite(hv).all()
    np.testing.assert_array_equal(hidx.cpu().numpy(), hi.numpy())
    zz = (hv[:, :, 0, :, None] + hv[:, :, 1, None, :]).reshape(T, H, -1)
    ii = (hi[:, :, 0, :, None] * S + hi[:, :, 1, None, :]).reshape(T, H, -1)
    ii, o = torch.sort(ii, dim=-1)  # equal sums: lower index first
    zz, o = torch.sort(torch.gather(zz, -1, o), dim=-1, descending=True, stable=True)
    np.testing.assert_array_equal(idx.cpu().numpy(), torch.gather(ii, -1, o)[..., :k].numpy())
    np.testing.assert_array_equal(h64(score), zz[..., :k].numpy())
    assert normwise(h64(w), torch.softmax(zz[..., :k], -1).numpy()) <= TOL_F32


@pytest.mark.parametrize("m", [0, 1, 5])
@pytest.mark.parametrize("S", [512, 2049])
def test_too_few_scores_that_are_numbers(gpu_lib, S, m):
    """A half with m < k such scores: the half lists go on with row 0 and every
    index lies in the table (it may be handed to the bag), on the path for few
    rows and on the one for many; with enough pairs left the selection is exact."""
    print(f"[too-few] {S} {m}", flush=True)
    H, d, k, T = 2, 32, 8, 4
    nan = torch.ones(S, dtype=torch.bool)
    nan[[S - 1, 7, S // 2, 64, 3][:m]] = False
    q, K, z = _with_nan_rows(S, H, d, T, nan, 421)
    order = torch.sort(z, dim=-1, descending=True, stable=True)
    hv, hi = order.values[..., :m], order.indices[..., :m]
    zz = (hv[:, :, 0, :, None] + hv[:, :, 1, None, :]).reshape(T, H, -1)
    ii = (hi[:, :, 0, :, None] * S + hi[:, :, 1, None, :]).reshape(T, H, -1)
    ii, o = torch.sort(ii, dim=-1)
    zz, o = torch.sort(torch.gather(zz, -1, o), dim=-1, descending=True, stable=True)
    want = torch.gather(ii, -1, o)[..., :k]
    for reps in (1, -(-(1 << 26) // (2 * T * H * S))):  # rows * S >= 2^26
        idx, w, score, hidx = pk.mem_search(q.cuda().repeat(reps, 1, 1), K.cuda(), k, want_half=True)
        torch.cuda.synchronize()
        idx, hidx = idx.cpu().view(reps, T, H, k), hidx.cpu().view(reps, T, H, 2, k)
        assert int(idx.min()) >= 0 and int(idx.max()) < S * S
        assert (hidx[..., :m] == hi).all() and (hidx[..., m:] == 0).all()
        c = want.shape[-1]  # pairs of two numbers among the k
        assert (idx[..., :c] == want).all()
