"""The reduction's loads that ask for no place in the caches (reads_once in csrc/fk_update.hip: X larger than the last-level
cache): a wave and a workgroup per item, rows of a cache line and wider ones, remainders of both."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,B,N,d,K", [
    (torch.float16, 1, 1100003, 128, 77), (torch.bfloat16, 3, 700001, 72, 300), (torch.float32, 1, 2200001, 32, 40),
    (torch.float16, 1, 4500001, 64, 33), (torch.float32, 2, 70003, 512, 9), (torch.bfloat16, 1, 300007, 504, 700),
])
def test_update_of_x_larger_than_the_caches(dtype, B, N, d, K):
    assert B * N * d * X_SIZE[dtype] > 1 << 28
    g = torch.Generator(device=DEV).manual_seed(N + d + K)
    X = torch.randn((B, N, d), generator=g, device=DEV).to(dtype)
    C0 = torch.randn((B, K, d), generator=g, device=DEV)
    label = (K * torch.rand((B, N), generator=g, device=DEV) ** 3).int().clamp_(max=K - 1)
    C, lp, n = fk.fk_update(X, label, C0)
    for b in range(B):
        at = label[b].long()
        total, size = (torch.zeros((K, d), dtype=torch.float64, device=DEV) for _ in range(2))
        for r in range(0, N, 1 << 16):
            x, member = X[b, r : r + (1 << 16)].double(), torch.nn.functional.one_hot(at[r : r + (1 << 16)], K).double().t()
            total += member @ x
            size += member @ x.abs()
        m = torch.bincount(at, minlength=K)
        assert torch.equal(n[b].long(), m)
        want = torch.where(m[:, None] > 0, total / m.clamp(min=1)[:, None], C0[b].double())
        # m additions of 2^-24 of the magnitudes' sum each at most, divided by m, and the rounded mean
        assert ((C[b].double() - want).abs() <= 2.0 ** -24 * (size + want.abs())).all()
    assert torch.equal(lp, C.to(dtype))


X_SIZE = {torch.float16: 2, torch.bfloat16: 2, torch.float32: 4}
