"""More clusters than one sort pass takes (K > 2048): ids up to the largest in 16 bits, points and clusters around the shares of
a workgroup of the boundary and item kernels (1024 each, csrc/fk_sort.hip), odd batch offsets, and the update over the tables."""
import numpy as np
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _labels(B, N, K, seed):
    g = torch.Generator().manual_seed(seed)
    a = torch.randint(0, K, (B, N), generator=g)
    a[torch.rand((B, N), generator=g) < 0.3] = K - 1        # the largest id, many items
    a[a == 1024] = 1023                                     # an empty cluster at a share's edge
    return a.to(torch.int32)


@pytest.mark.parametrize("B,N,K", [(1, 1, 65536), (3, 1023, 2049), (3, 1025, 65536), (1, 4096, 3072), (3, 4097, 65535), (1, 70001, 3073),
                                   (2, 50001, 65536)])
def test_sort_with_many_clusters(B, N, K):
    a = _labels(B, N, K, N + K)
    idx, off = fk.fk_sort_inverse(a.to(DEV), K)
    for b in range(B):
        assert np.array_equal(idx[b].cpu().numpy(), np.argsort(a[b].numpy(), kind="stable"))
        assert off[b].tolist() == [0] + torch.bincount(a[b], minlength=K).cumsum(0).tolist()


@pytest.mark.parametrize("B,N,d,K", [(2, 30001, 16, 2049), (1, 50000, 24, 3072), (1, 50000, 24, 3073), (2, 40001, 8, 65536)])
def test_update_with_many_clusters(B, N, d, K):
    a = _labels(B, N, K, N)
    g = torch.Generator().manual_seed(K)
    X = torch.randn((B, N, d), generator=g).half()
    C0 = torch.randn((B, K, d), generator=g)
    C, _, n = fk.fk_update(X.to(DEV), a.to(DEV), C0.to(DEV))
    for b in range(B):
        cnt = torch.bincount(a[b], minlength=K)
        assert torch.equal(n[b].cpu().long(), cnt)
        s = torch.zeros((K, d), dtype=torch.float64).index_add_(0, a[b].long(), X[b].double())
        ref = torch.where(cnt[:, None] > 0, s / cnt.clamp(min=1)[:, None], C0[b].double())
        size = torch.zeros((K, d), dtype=torch.float64).index_add_(0, a[b].long(), X[b].double().abs()) / cnt.clamp(min=1)[:, None]
        # sums of n terms: at most n 2^-24 of their sizes' sum, and one rounding each of 1 / n and of the product
        assert ((C[b].cpu().double() - ref).abs() <= (cnt[:, None] + 3) * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,N,d,K,rows", [(1, 9000, 8, 4097, 1), (1, 20001, 128, 4099, 3), (2, 30000, 16, 2051, 300), (32, 700, 40, 37, 1),
                                          (33, 2000, 104, 34, 1), (16, 5000, 128, 70, 1)])
def test_merge_by_a_wave_per_cluster(dtype, B, N, d, K, rows):
    """Many clusters of few partial rows (finalize_wave_kernel), some empty, one with `rows` rows in every ten; the fit's next
    iteration multiplies what the merge laid out, so that it must give a new call's assignment."""
    g = torch.Generator().manual_seed(N + d + K)
    a = torch.randint(0, K, (B, N), generator=g)
    a[torch.rand((B, N), generator=g) < rows / (rows + 10.0)] = K // 2
    a[a == K - 1] = 0
    X = torch.randn((B, N, d), generator=g).to(dtype)
    C0 = torch.randn((B, K, d), generator=g)
    C, lp, n = fk.fk_update(X.to(DEV), a.int().to(DEV), C0.to(DEV))
    assert torch.equal(lp.cpu(), C.cpu().to(dtype))
    for b in range(0, B, 7):
        cnt = torch.bincount(a[b], minlength=K)
        assert torch.equal(n[b].cpu().long(), cnt)
        assert torch.equal(C[b, K - 1].cpu(), C0[b, K - 1])
        s = torch.zeros((K, d), dtype=torch.float64).index_add_(0, a[b], X[b].double())
        size = torch.zeros((K, d), dtype=torch.float64).index_add_(0, a[b], X[b].double().abs()) / cnt.clamp(min=1)[:, None]
        ref = torch.where(cnt[:, None] > 0, s / cnt.clamp(min=1)[:, None], C0[b].double())
        assert ((C[b].cpu().double() - ref).abs() <= (cnt[:, None] + 3) * 2.0 ** -24 * size).all()
    two, one = C0.to(DEV), C0.to(DEV)
    a2, n2, _ = fk.fk_lloyd_iter(X.to(DEV), two, 2)
    fk.fk_lloyd_iter(X.to(DEV), one, 1)
    a1, n1, _ = fk.fk_lloyd_iter(X.to(DEV), one, 1)
    assert torch.equal(a2, a1) and torch.equal(n2, n1) and torch.equal(two, one)


@pytest.mark.parametrize("dtype,N,d,K", [(torch.float32, 20000, 16, 1500), (torch.float32, 30000, 33, 1200), (torch.float16, 20000, 9, 900),
                                         (torch.float32, 60000, 8, 3000)])
def test_merge_adds_in_one_order(dtype, N, d, K):
    """Clusters of several partial rows: rows as stored and padded ones, and three iterations in one call and in three (where the
    merges before a call's last may write split centroids by another kernel), give the same bits."""
    g = torch.Generator().manual_seed(N + d)
    size = torch.rand((K,), generator=g) ** 6               # a few large clusters
    lab = torch.multinomial(size + 1e-3, N, replacement=True, generator=g)
    centre = 8 * torch.randn((K, d), generator=g)
    X = (centre[lab] + torch.randn((N, d), generator=g)).to(dtype)[None].to(DEV)
    C0 = centre[None].to(DEV)
    pad = -d % 8
    three, steps, padded = C0.clone(), C0.clone(), torch.nn.functional.pad(C0, (0, pad))
    fk.fk_lloyd_iter(X, three, 3)
    for _ in range(3):
        fk.fk_lloyd_iter(X, steps, 1)
    fk.fk_lloyd_iter(torch.nn.functional.pad(X, (0, pad)), padded, 3)
    assert torch.equal(three, steps) and torch.equal(three, padded[..., :d])
