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
    # rows as they are stored, that are no multiple of 8
    (1, 129, 100, 300), (2, 65, 63, 70), (1, 200, 250, 130), (1, 40, 500, 70), (1, 33, 9, 40),
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
            if d % 8 == 0:
                res.append(fk.fk_assign_static(X, C, min_dist=True))
    finally:
        fk.fk_set_option("assign_few", -1)
    for a, m in res[1:]:
        assert torch.equal(a, res[0][0]) and torch.equal(m, res[0][1])


@pytest.mark.parametrize("B,N,d,K,few", [
    # around the lines of the rule (256 compute units): tiles of centroids, chunks of features, points
    (1, 1000, 136, 40, True), (1, 128, 320, 40, False), (1, 129, 320, 40, True), (1, 1, 512, 96, True), (1, 1, 512, 64, False),
    (1, 1, 512, 97, True), (1, 8193, 136, 64, False), (1, 8193, 136, 65, True), (1, 8193, 192, 40, True), (1, 8193, 264, 224, False),
    (1, 8193, 264, 225, True), (1, 8192, 128, 1024, True), (1, 65536, 128, 1024, False),
])
def test_the_rule_takes_it_where_it_is_faster_and_answers_alike(B, N, d, K, few):
    g = torch.Generator(device=DEV).manual_seed(N + d + K)
    X, C = (torch.randn((B, n, d), generator=g, device=DEV).half() for n in (N, K))
    assert ("mfma_few" in fk.fk_plan(B, N, d, K, torch.float16)) == few
    a, m = fk.fk_assign(X, C, min_dist=True)
    try:
        fk.fk_set_option("assign_few", 0)
        b, n = fk.fk_assign(X, C, min_dist=True)
        c = C.float()
        u = fk.fk_lloyd_iter(X, c, 1)
        fk.fk_set_option("assign_few", -1)
        e = C.float()
        v = fk.fk_lloyd_iter(X, e, 1)
    finally:
        fk.fk_set_option("assign_few", -1)
    assert torch.equal(a, b) and torch.equal(m, n)
    assert torch.equal(u[0], v[0]) and torch.equal(c, e)
