"""The one-pass update for few clusters (stream_update_kernel in csrc/fk_fused.hip) around the ends of its batches of 32
points, of its waves' and its workgroups' shares, and with widths that fill a chunk, a row piece or neither."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("d", [5, 8, 24, 32, 40, 64, 72, 100, 128])
@pytest.mark.parametrize("B,N,K", [
    (1, 1, 1), (1, 31, 2), (2, 33, 3), (1, 127, 32), (3, 129, 17), (1, 4096, 31), (1, 32769, 32), (1, 65569, 9), (300, 65, 5),
])
def test_few_cluster_batches(dtype, B, N, d, K):
    g = torch.Generator(device=DEV).manual_seed(N + d + K)
    centre = 8 * torch.randn((B, K, d), generator=g, device=DEV)
    label = torch.randint(0, K, (B, N), generator=g, device=DEV)
    x = centre.gather(1, label[..., None].expand(B, N, d)) + 0.05 * torch.randn((B, N, d), generator=g, device=DEV)
    X, C0 = x.to(dtype), centre.to(dtype).float()
    # (components may lie close together in a few dimensions: the nearest one, not the one drawn)
    label = torch.cdist(X.double(), C0.double(), compute_mode="donot_use_mm_for_euclid_dist").argmin(-1)
    hot = torch.nn.functional.one_hot(label, K).double().transpose(1, 2)
    n = hot.sum(-1)
    total, size = hot @ X.double(), hot @ X.double().abs()
    want = torch.where(n[..., None] > 0, total / n.clamp(min=1)[..., None], C0.double())
    # n additions in the matrix pipe, 2^-23 of the magnitudes' sum each at most, divided by n; and the rounded mean
    bound = 2.0 ** -23 * (size + want.abs())
    C = C0.clone()
    a, m, lp = fk.fk_lloyd_iter(X, C, 1)
    assert torch.equal(a.long(), label) and torch.equal(m.double(), n)
    assert ((C.double() - want).abs() <= bound).all()
    assert torch.equal(lp, C.to(dtype))
    D, lp, m = fk.fk_update(X, label.int(), C0)
    assert torch.equal(m.double(), n) and ((D.double() - want).abs() <= bound).all() and torch.equal(lp, D.to(dtype))
    # only the last iteration of a call leaves its assignment; three calls of one leave the same bits
    three, ones = C0.clone(), C0.clone()
    a = torch.full((B, N), -7, dtype=torch.int32, device=DEV)
    fk.fk_lloyd_iter(X, three, 3, assign=a)
    for _ in range(3):
        b, _, _ = fk.fk_lloyd_iter(X, ones, 1)
    assert torch.equal(a, b) and torch.equal(three, ones)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("B,N,d,few", [(1, 1 << 24, 64, 11), (1, (1 << 24) - 45, 40, 11), (2, (1 << 23) - 3, 24, 12), (1, 1 << 23, 128, 12)])
def test_long_chains(dtype, B, N, d, few):
    """Of sixteen points of a batch 15 are ones and one is 3/4 of half a place of a sum of half the points that a wave adds up: one chain
    over all of them drops it there, 5 to 12 parts in 10^6 of the mean."""
    small = 0.75 * 2.0 ** -few
    X = torch.ones((B, N, d), dtype=dtype, device=DEV)
    X[:, 5::16] = small
    want = 1 + (small - 1) * len(range(5, N, 16)) / N
    # Small values are multiples of 2^-(few + 2) and a run of 32 batches adds up to less than 2^10; whole runs are multiples of 2^(4 - few)
    # and a workgroup's add up to 2^(27 - few) at the most: all exact.  What rounds is what ends a wave's share, the four waves' sums where
    # N is ragged, fewer than 34 additions of positive numbers in the merge, its division and the conversion.
    bound = 42 * 2.0 ** -24
    C0 = torch.full((B, 2, d), -5.0, device=DEV)
    C0[:, 0] = 1.0
    C, _, n = fk.fk_update(X, torch.zeros((B, N), dtype=torch.int32, device=DEV), C0)
    assert n.tolist() == [[N, 0]] * B
    assert ((C[:, 0].double() / want - 1).abs() <= bound).all()
    if d > 64:
        return               # (the fit has no registers for a second level there; its chains are as they always were)
    C = C0.clone()
    _, n, _ = fk.fk_lloyd_iter(X, C, 1)
    assert n.tolist() == [[N, 0]] * B
    assert ((C[:, 0].double() / want - 1).abs() <= bound).all()
