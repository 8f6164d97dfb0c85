"""Rows of more than 128 16-bit features around the lines between the few-point form, workgroups of four waves and of eight
(choose_few and launch_mfma_wide in csrc/fk_assign.hip): the same bits whichever takes them."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("d", [136, 200, 256, 300, 384, 512])
@pytest.mark.parametrize("B,N,K", [(1, 16385, 40), (1, 24576, 300), (1, 24577, 1030), (1, 32769, 300), (5, 6500, 70), (3, 11001, 1030)])
def test_wide_rows_give_the_same_bits_on_every_route(dtype, d, B, N, K):
    g = torch.Generator(device=DEV).manual_seed(N + d + K)
    X = torch.randn((B, N, d), generator=g, device=DEV).to(dtype)
    C = torch.randn((B, K, d), generator=g, device=DEV).to(dtype)
    got = []
    try:
        for form in (-1, 0, 2):                  # by shape, sweeping, one tile of points to a workgroup
            fk.fk_set_option("assign_few", form)
            got.append(fk.fk_assign(X, C, min_dist=True))
    finally:
        fk.fk_set_option("assign_few", -1)
    for a, m in got[1:]:
        assert torch.equal(a, got[0][0]) and torch.equal(m, got[0][1])
    step = 1 << 12                               # the nearest by the stored values, up to the comparison at 2^-19 of a score
    for b in range(B):
        c = C[b].double()
        for r in range(0, N, step):
            D = torch.cdist(X[b, r : r + step].double(), c).square()
            mine = D.gather(1, got[0][0][b, r : r + step, None].long())[:, 0]
            assert (mine <= D.min(1).values + 2.0 ** -17 * (c.square().sum(1).max() + D.max())).all()
