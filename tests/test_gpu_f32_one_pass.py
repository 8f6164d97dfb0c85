"""The one-pass update of small fp32 problems (csrc/fk_f32_fused.hip) in four, eight and sixteen waves, on rows that
end in a whole piece of 16, in half of one and inside one: the general path's assignments and counts."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,N", [(1, 15), (2, 1000), (1, 16384), (1, 16449), (7, 2500)])
@pytest.mark.parametrize("d,K", [(9, 4), (16, 5), (24, 9), (30, 64), (33, 4), (40, 17), (64, 16), (64, 17), (63, 64), (72, 8), (100, 9), (121, 64), (128, 33)])
def test_one_pass_equals_the_general_path(B, N, d, K):
    K = min(K, N)
    g = torch.Generator(device=DEV).manual_seed(N + d + K)
    X = torch.randn((B, N, d), generator=g, device=DEV)
    res = []
    try:
        for v in (-1, 0):
            fk.fk_set_option("fused_update", v)
            fk.fk_set_option("gather_update", v)
            assert ("f32_update" in fk.fk_plan(B, N, d, K, torch.float32)) == (v < 0)
            C = X[:, :K].clone()
            a, n, _ = fk.fk_lloyd_iter(X, C, 1)
            res.append((a, n, C))
    finally:
        fk.fk_set_option("fused_update", -1)
        fk.fk_set_option("gather_update", -1)
    (a, n, C), (b, m, D) = res
    assert torch.equal(a, b) and torch.equal(n, m)
    # the same n terms in two orders: n 2^-24 of their largest each, divided by n
    assert ((C - D).abs() <= 2 * 2.0 ** -24 * n.amax() * X.abs().amax()).all()
