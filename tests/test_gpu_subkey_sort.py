"""The search backward's counting sort at the sizes where its form changes: the
first size past the one-workgroup sort (8192 slots), token tiles of 16 and more
and their remainders, sub-key numbers around multiples of 256, tables that only
larger tiles or only the radix sort take (few lookups of many sub-keys), k up to
64, sub-keys of more than 2048 tokens, rows without any lookup.

Small integer gradients and queries make every sum an exact integer in fp32
whatever its order, so the sub-key gradients must equal the reference exactly."""
import pytest
import torch

import paper_2412_09764_amd as pk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,S,k,hot", [
    (4096, 1, 1, 1, 0), (4097, 1, 1, 1, 0), (257, 1, 3, 17, 0), (129, 1, 255, 32, 0.5),
    (130, 4, 256, 33, 0), (131, 3, 257, 64, 0), (2500, 2, 700, 5, 0.9), (8192, 1, 8192, 1, 0),
    (8191, 1, 8192, 1, 0), (300, 4, 8192, 32, 0), (255, 4, 8192, 32, 0), (9000, 2, 64, 8, 0.3),
    (33000, 4, 130, 2, 0),
])
def test_subkey_gradients_exact(gpu_lib, T, H, S, k, hot):
    print(f"[subkey-sort] {T} {H} {S} {k} {hot}", flush=True)
    d = 8
    g = torch.Generator().manual_seed(91 + T)
    idx = torch.randint(0, S * S, (T, H, k), generator=g)
    if hot:
        idx[torch.rand((T, H, k), generator=g) < hot] = S * S - 1
    idx[torch.rand((T, H, 1), generator=g).expand(T, H, k) < 0.1] = -1  # whole rows absent
    idx = idx.cuda()
    q = torch.randint(-2, 3, (T, H, 2 * d), generator=g).to(torch.bfloat16).cuda()
    K = torch.zeros((H, 2, S, d), dtype=torch.bfloat16, device="cuda")
    gz = torch.randint(-2, 3, (T, H, k), generator=g).float().cuda()
    base = torch.randint(-5, 6, (H, 2, S, d), generator=g).float().cuda()
    _, gK = pk.mem_search_backward(q, K, idx, gz, grad_subkeys=base.clone(), want_grad_q=False)
    torch.cuda.synchronize()
    want = base.double()
    live, safe = (gz * (idx >= 0)).double(), idx.clamp(min=0)
    for p, i in enumerate((safe // S, safe % S)):
        for h in range(H):
            src = live[:, h, :, None] * q[:, h, None, p * d:(p + 1) * d].double()
            want[h, p].index_add_(0, i[:, h].reshape(-1), src.reshape(-1, d))
    assert torch.equal(gK.double(), want)


@pytest.mark.parametrize("T,H,S,k", [
    (520, 1, 1024, 8), (520, 1, 1026, 8),            # tiles of 64 tokens; 128 of them: radix
    (32768, 2, 2048, 8), (32767, 2, 2048, 8),        # tiles of 128 from 2^20 slots up
    (33000, 2, 4100, 8), (4097, 1, 8192, 2),         # tiles of more: radix, in three launches and chained
])
def test_subkey_gradients_at_the_rule(gpu_lib, T, H, S, k):
    """Both sorts at the lines of the rule that chooses between them."""
    test_subkey_gradients_exact(gpu_lib, T, H, S, k, 0.05)
