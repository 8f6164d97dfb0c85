"""Few points against many centroids (assign_mfma_few_kernel): every form gives the sweeping kernels' bits."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("B,N,d,K", [
    (1, 1, 8, 1), (1, 31, 24, 33), (2, 33, 32, 17 * 32 + 1), (1, 65, 40, 512), (3, 100, 64, 100),
    (1, 64, 96, 1025), (1, 1000, 128, 1024), (1, 97, 136, 300), (2, 63, 256, 64), (1, 200, 264, 129), (1, 70, 512, 95),
])
def test_every_form_gives_the_sweeping_kernels_answer(dtype, B, N, d, K):
    g = torch.Generator().manual_seed(N + d + K)
    X = (4 * torch.randn((B, N, d), generator=g)).to(dtype).to(DEV)
    C = (4 * torch.randn((B, K, d), generator=g)).to(dtype).to(DEV)
    C[:, K // 2] = C[:, 0]                       # an exact tie
    X[:, N // 2] = C[:, 0]
    res = []
    try:
        for v in (0, 1, 2, 3, 4):
            fk.fk_set_option("assign_few", v)
            assert ("mfma_few" in fk.fk_plan(B, N, d, K, dtype)) == (v > 0)
            res.append(fk.fk_assign(X, C, min_dist=True))
            res.append(fk.fk_assign_static(X, C, min_dist=True))
    finally:
        fk.fk_set_option("assign_few", -1)
    for a, m in res[1:]:
        assert torch.equal(a, res[0][0]) and torch.equal(m, res[0][1])
