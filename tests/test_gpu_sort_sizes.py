"""The backwards' sort at the sizes where its form changes: one workgroup up to
8192 keys, a chain of passes up to 2^19, three launches per pass beyond; tiles
of 4096 keys; one to four radix passes; rows of slots of which only some are
filled; skewed keys (one hot row).

Small integer weights, gradients and queries make every sum an exact integer in
fp32 whatever its order, so results must equal the references exactly."""
import pytest
import torch

import paper_2412_09764_amd as pk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,hot", [
    (1, 5, 0), (63, 200, 0), (1025, 300, 0), (8191, 70000, 0), (8192, 1 << 16, 0.5),
    (8193, 1 << 16, 0), (12288, 1 << 20, 0.3), (20000, (1 << 24) + 5, 0), (65536, 200, 0),
    (1 << 19, 1 << 18, 0.2), ((1 << 19) + 1, 1 << 18, 0),
])
def test_value_backward_sort_sizes(gpu_lib, T, N, hot):
    print(f"[sort-sizes] {T} {N} {hot}", flush=True)
    D = 8
    g = torch.Generator().manual_seed(31 + T)
    idx = torch.randint(0, N, (T, 1, 1), generator=g)
    if hot:
        idx[torch.rand(T, generator=g) < hot] = N // 3
    idx = idx.cuda()
    w = torch.randint(-2, 3, (T, 1, 1), generator=g).float().cuda()
    dy = torch.randint(-2, 3, (T, D), generator=g).to(torch.bfloat16).cuda()
    V = torch.randint(-2, 3, (1, D), generator=g).to(torch.bfloat16).cuda().expand(N, D).contiguous()
    rows, grows, gw, _ = pk.mem_bag_backward_sparse(dy, V, idx, w)
    torch.cuda.synchronize()
    want, inv = torch.unique(idx.reshape(-1), return_inverse=True)
    ref = torch.zeros((want.numel(), D), dtype=torch.float64, device="cuda")
    ref.index_add_(0, inv, (w.reshape(T, 1) * dy.float()).double())
    assert torch.equal(rows, want)
    assert torch.equal(grows.double(), ref)
    assert torch.equal(gw.reshape(T), (dy.float() * V[0].float()).sum(1))


@pytest.mark.parametrize("T,H,S,k,hot", [
    (1, 1, 3, 1, 0), (7, 2, 64, 9, 0), (128, 1, 1000, 32, 0), (129, 1, 70, 32, 0.5),
    (300, 2, 2048, 32, 0), (2048, 4, 512, 32, 0.9), (2049, 4, 512, 32, 0), (3000, 3, 8192, 20, 0),
])
def test_search_backward_sort_sizes(gpu_lib, T, H, S, k, hot):
    print(f"[sbwd-sizes] {T} {H} {S} {k} {hot}", flush=True)
    d = 8
    g = torch.Generator().manual_seed(57 + T)
    idx = torch.randint(0, S * S, (T, H, k), generator=g)
    idx[torch.rand((T, H, k), generator=g) < 0.1] = -1  # absent: contributes nothing
    if hot:
        idx[torch.rand((T, H, k), generator=g) < hot] = S + 1
    idx = idx.cuda()
    q = torch.randint(-2, 3, (T, H, 2 * d), generator=g).to(torch.bfloat16).cuda()
    K = torch.randint(-2, 3, (H, 2, S, d), generator=g).to(torch.bfloat16).cuda()
    gz = torch.randint(-2, 3, (T, H, k), generator=g).float().cuda()
    gq, gK = pk.mem_search_backward(q, K, idx, gz)
    torch.cuda.synchronize()
    rq = torch.zeros_like(gq, dtype=torch.float64)
    rK = torch.zeros_like(gK, dtype=torch.float64)
    live = gz * (idx >= 0)
    safe = idx.clamp(min=0)
    for p, i in enumerate((safe // S, safe % S)):
        for h in range(H):
            rows = K[h, p][i[:, h]].double()  # [T, k, d]
            rq[:, h, p * d:(p + 1) * d] = (live[:, h, :, None].double() * rows).sum(1)
            src = live[:, h, :, None].double() * q[:, h, None, p * d:(p + 1) * d].double()
            rK[h, p].index_add_(0, i[:, h].reshape(-1), src.reshape(-1, d))
    assert torch.equal(gq.double(), rq)
    assert torch.equal(gK.double(), rK)


@pytest.mark.parametrize("T,H,S,k", [(29, 512, 8192, 32), (40, 512, 8192, 32), (43, 300, 8190, 41)])
def test_search_backward_of_many_heads(gpu_lib, T, H, S, k):
    """Slots of many heads and few tokens, too few to count per sub-key: the
    chain of passes up to 2^20 of them, three launches a pass beyond; rows of
    which only some slots are filled, and some of none."""
    print(f"[sbwd-heads] {T} {H} {S} {k} {2 * T * H * k}", flush=True)
    d = 8
    g = torch.Generator(device="cuda").manual_seed(77 + T)
    idx = torch.randint(0, S * S, (T, H, k), generator=g, device="cuda")
    idx[torch.rand((T, H, k), generator=g, device="cuda") < 0.3] = 5 * S + 3  # shared sub-keys
    idx[torch.rand((T, H, 1), generator=g, device="cuda").expand(T, H, k) < 0.1] = -1
    q = torch.randint(-2, 3, (T, H, 2 * d), generator=g, device="cuda").to(torch.bfloat16)
    K = torch.zeros((H, 2, S, d), dtype=torch.bfloat16, device="cuda")
    gz = torch.randint(-2, 3, (T, H, k), generator=g, device="cuda").float()
    _, gK = pk.mem_search_backward(q, K, idx, gz, want_grad_q=False)
    torch.cuda.synchronize()
    want = torch.zeros((H * 2 * S, d), dtype=torch.float32, device="cuda")  # whole numbers: exact
    live, safe = gz * (idx >= 0), idx.clamp(min=0)
    heads = torch.arange(H, device="cuda")[None, :, None]
    for p, i in enumerate((safe // S, safe % S)):
        src = live[..., None] * q[:, :, None, p * d:(p + 1) * d].float()
        want.index_add_(0, ((heads * 2 + p) * S + i).reshape(-1), src.reshape(-1, d))
    assert torch.equal(gK.reshape(-1, d), want)
