"""fp32 fits through the matrix-core filter whose updates write the next assignment's split centroids (emit_split in
csrc/fk_update.hip): the bits of calls of one iteration each, which lay them out anew, and of the direct kernels, with and without a
sort, for ragged rows, several instances, clusters without points, and rows that are not finite or whose squares overflow."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("odd", [None, float("nan"), float("inf"), 3e19])
@pytest.mark.parametrize("gather", [-1, 0, 1, 2])
@pytest.mark.parametrize("B,N,d,K", [(1, 3001, 100, 33), (2, 5000, 44, 130), (1, 9000, 256, 40), (3, 1200, 512, 31), (1, 40000, 96, 300),
                                     (1, 2000, 7, 200), (1, 30000, 129, 64)])
def test_fit_equals_single_iterations(odd, gather, B, N, d, K):
    g = torch.Generator(device=DEV).manual_seed(N + d + K)
    centre = 5 * torch.randn((B, K, d), generator=g, device=DEV) + 3
    X = centre.gather(1, torch.randint(0, K, (B, N, 1), generator=g, device=DEV).expand(B, N, d)) + torch.randn((B, N, d), generator=g, device=DEV)
    C0 = X[:, :K].contiguous()
    C0[:, 1] = 500.0                             # a cluster without points: it keeps its centroid
    if odd is not None:
        C0[:, K // 2, d - 1] = odd
    got = []
    try:
        fk.fk_set_option("fused_update", 0)
        fk.fk_set_option("gather_update", gather)
        for option in (1, 0):
            fk.fk_set_option("assign_f32_filter", option)
            whole, ones = C0.clone(), C0.clone()
            a, n, lp = fk.fk_lloyd_iter(X, whole, 4)
            for _ in range(4):
                b, m, _ = fk.fk_lloyd_iter(X, ones, 1)
            assert torch.equal(a, b) and torch.equal(n, m)
            assert torch.equal(whole.view(torch.int32), ones.view(torch.int32)) and torch.equal(lp.view(torch.int32), whole.view(torch.int32))
            got.append((a, n, whole))
    finally:
        for name in ("assign_f32_filter", "gather_update", "fused_update"):
            fk.fk_set_option(name, -1)
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert torch.equal(got[0][2].view(torch.int32), got[1][2].view(torch.int32))
