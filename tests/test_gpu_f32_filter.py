"""fp32 assignment through the matrix-core filter (csrc/fk_f32_filter.hip): the same bits as the direct
fp32 kernels, whatever the data -- the filter may only decide points whose answer no rounding can
change, everything else is measured by the direct kernels' arithmetic."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture
def both():
    """Assignments (and distances) of the filtered and of the direct kernels."""
    def run(X, C):
        res = []
        for v in (1, 0):
            fk.fk_set_option("assign_f32_filter", v)
            assert ("f32_filter" in fk.fk_plan(X.shape[0], X.shape[1], X.shape[2], C.shape[1], X.dtype)) == (v == 1)
            res.append(fk.fk_assign(X, C, min_dist=True))
        return res
    yield run
    fk.fk_set_option("assign_f32_filter", -1)


def _data(kind, B, N, d, K, seed):
    g = torch.Generator().manual_seed(seed)
    X = torch.randn((B, N, d), generator=g)
    pick = torch.stack([torch.randint(0, N, (K,), generator=g) for _ in range(B)])
    if kind == "mixture":
        X += 4 * torch.randn((B, K, d), generator=g).gather(1, torch.randint(0, K, (B, N, 1), generator=g).expand(B, N, d))
    elif kind == "far":             # a common offset far larger than the spread
        X += 1000.0
    elif kind == "whole":           # exact ties: small whole numbers
        X = torch.randint(-2, 3, (B, N, d), generator=g).float()
    elif kind == "large":           # squares near and beyond the end of the range
        X *= 3e18
    elif kind == "small":           # squares that vanish
        X *= 1e-21
    C = torch.stack([X[b, pick[b]] for b in range(B)])
    if kind == "twins":             # every centroid twice
        C = torch.cat([C[:, : (K + 1) // 2]] * 2, 1)[:, :K]
    elif kind == "triples":
        C = torch.cat([C[:, : (K + 2) // 3]] * 3, 1)[:, :K]
    elif kind == "border":          # between two centroids, 2^-4 .. 2^-28 of their distance off the middle
        C[:, 1::2] = C[:, : K // 2 * 2 : 2] + 0.1 * torch.randn(C[:, 1::2].shape, generator=g)
        of = torch.randint(0, max(1, K // 2), (B, N, 1), generator=g).expand(B, N, d) * 2
        u, v = C.gather(1, of), C.gather(1, (of + 1).clamp(max=K - 1))
        off = torch.exp2(-4 - 24 * torch.rand((B, N, 1), generator=g)) * (torch.randint(0, 2, (B, N, 1), generator=g) * 2 - 1)
        X = (u + v) * 0.5 + off * (v - u)
    elif kind == "outlier":         # one centroid far away, the first
        C[:, 0] = 1e6
    return X.to(DEV), C.contiguous().to(DEV)


@pytest.mark.parametrize("kind", ["gauss", "mixture", "far", "whole", "large", "small", "twins", "triples", "border", "outlier"])
@pytest.mark.parametrize("B,N,d,K", [(1, 3001, 64, 100), (2, 517, 8, 33), (1, 1000, 96, 257), (1, 4100, 128, 64),
                                     (1, 700, 256, 97), (1, 300, 512, 70), (3, 130, 32, 1), (1, 333, 392, 31)])
def test_filter_gives_the_direct_answer(both, kind, B, N, d, K):
    X, C = _data(kind, B, N, d, K, seed=N + d + K)
    (a1, m1), (a0, m0) = both(X, C)
    assert torch.equal(a1, a0)
    # the distances are sums of d squares in two orders: d 2^-23 apart at most
    fine = torch.isfinite(m0)
    assert torch.equal(fine, torch.isfinite(m1))
    assert ((m1 - m0).abs()[fine] <= d * 2.0 ** -23 * m0[fine] + 1e-37).all()


@pytest.mark.parametrize("kind,B,N,d,K", [
    # many open points: a thread each (rows of up to 32 and 64, few and many centroids), P = 8 with one team and
    # with as many as there is room for; more points than four waves take
    ("twins", 1, 140000, 32, 64), ("twins", 1, 140000, 60, 100), ("triples", 1, 133000, 48, 300), ("twins", 1, 3000, 64, 300),
    ("twins", 1, 9001, 500, 100), ("twins", 1, 20001, 128, 64), ("mixture", 1, (1 << 19) + 5, 40, 30), ("border", 1, (1 << 19) + 5, 100, 50),
])
def test_filter_gives_the_direct_answer_for_many_points(both, kind, B, N, d, K):
    (a1, m1), (a0, m0) = both(*_data(kind, B, N, d, K, seed=N + d + K))
    assert torch.equal(a1, a0)
    assert ((m1 - m0).abs() <= d * 2.0 ** -23 * m0 + 1e-37).all()


@pytest.mark.parametrize("d", [7, 16, 32, 48, 61, 80, 96, 112, 128, 129, 160, 161, 192, 224, 256, 257, 320, 384, 448, 512])
@pytest.mark.parametrize("K", [1, 32, 33, 65, 300])
def test_every_number_of_chunks_with_few_and_many_tiles(both, d, K):
    """One stage, an odd and an even number of them, whole and half tiles per stage."""
    for kind in ("mixture", "whole"):
        (a1, m1), (a0, m0) = both(*_data(kind, 1, 777, d, K, seed=d + K))
        assert torch.equal(a1, a0)
        assert ((m1 - m0).abs() <= d * 2.0 ** -23 * m0 + 1e-37).all()


@pytest.mark.parametrize("N,d,K", [(3001, 64, 100), (1000, 96, 257), (700, 256, 97), (263000, 24, 40)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_what_is_not_finite_is_answered_as_by_the_direct_kernels(both, N, d, K, bad):
    g = torch.Generator().manual_seed(N + d)
    X = torch.randn((1, N, d), generator=g)
    C = X[:, :K].clone()
    X[0, N // 2, d // 2] = bad
    C[0, 3, d - 1] = bad
    C[0, K // 2] = bad
    for x, c in ((X, X[:, :K]), (X, C), (C, C), (C, torch.full_like(C, bad))):
        (a1, m1), (a0, m0) = both(x.to(DEV), c.contiguous().to(DEV))
        assert torch.equal(a1, a0)
        assert not m1.isnan().any() and torch.equal(m1.isinf(), m0.isinf())
        fine = m0.isfinite()
        assert ((m1 - m0).abs()[fine] <= d * 2.0 ** -23 * m0[fine] + 1e-37).all()


def test_distances_of_more_points_than_one_launch_dimension_has_threads_for(both):
    """2^28 points at 16 threads a point are 2^32 threads: the distance pass takes several groups each."""
    N = (1 << 28) + 5
    g = torch.Generator(device=DEV).manual_seed(3)
    X = torch.empty((1, N, 8), device=DEV).normal_(generator=g)
    C = X[:, :24].clone()
    (a1, m1), (a0, m0) = both(X, C)
    assert torch.equal(a1, a0)
    m1 -= m0
    assert (m1.abs_() <= m0.mul_(8 * 2.0 ** -23).add_(1e-37)).all()


def test_filtered_iterations_equal_direct_ones():
    g = torch.Generator().manual_seed(5)
    X = (torch.randn((2, 20011, 100), generator=g) + 3 * torch.randn((2, 1, 100), generator=g)).to(DEV)
    res = []
    try:
        for v in (1, 0):
            fk.fk_set_option("assign_f32_filter", v)
            C = X[:, :150].clone()
            a, n, _ = fk.fk_lloyd_iter(X, C, 3)
            res.append((a, n, C))
    finally:
        fk.fk_set_option("assign_f32_filter", -1)
    for u, v in zip(*res):
        assert torch.equal(u, v)
