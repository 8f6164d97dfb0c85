"""fp32 assignment of few points (assign_f32_filter_few_kernel in csrc/fk_f32_filter.hip) and points that are open between two
centroids: the bits of the direct kernels, around tiles of points, waves without a centroid tile, the line to the sweep, and the
lists of both kinds in one call."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk
from tests.test_gpu_f32_filter import _data, both  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def _same(both, X, C):
    (a1, m1), (a0, m0) = both(X, C)
    assert torch.equal(a1, a0)
    # the distances are sums of d squares in two orders: d 2^-23 apart at most
    fine = torch.isfinite(m0)
    assert torch.equal(fine, torch.isfinite(m1))
    assert ((m1 - m0).abs()[fine] <= X.shape[2] * 2.0 ** -23 * m0[fine] + 1e-37).all()
    fk.fk_set_option("assign_f32_filter", 1)
    assert torch.equal(fk.fk_assign(X, C), a0)          # without distances the two centroids wait elsewhere


@pytest.mark.parametrize("kind", ["gauss", "whole", "twins", "border"])
@pytest.mark.parametrize("d", [5, 16, 32, 44, 64, 80, 96, 112, 128, 152, 192, 217, 256, 320, 384, 448, 512])
@pytest.mark.parametrize("B,N,K", [(1, 1, 1), (1, 31, 300), (3, 33, 64), (1, 641, 257), (2, 4095, 97)])
def test_few_points(both, kind, d, B, N, K):  # noqa: F811
    _same(both, *_data(kind, B, N, d, min(K, N) if kind != "gauss" else K, seed=N + d + K))


@pytest.mark.parametrize("kind", ["mixture", "twins", "triples", "border", "large", "small", "far"])
@pytest.mark.parametrize("B,N,d,K", [(1, 8192, 100, 40), (1, 8193, 100, 40), (1, 8193, 128, 128), (1, 16384, 256, 100), (1, 16385, 256, 100),
                                     (7, 2400, 264, 300), (1, 40001, 512, 290), (1, 30000, 130, 1100)])
def test_on_both_sides_of_the_line_and_with_both_lists(both, kind, B, N, d, K):  # noqa: F811
    _same(both, *_data(kind, B, N, d, K, seed=N + d + K))


@pytest.mark.parametrize("kind,d", [("twins", 72), ("twins", 93), ("twins", 48), ("triples", 200), ("triples", 509)])
@pytest.mark.parametrize("B,N,K", [(1, 8191, 300), (1, 8192, 270), (1, 16384, 400), (1, 32767, 130), (1, 32773, 300), (2, 16390, 100)])
def test_long_lists(both, kind, d, B, N, K):  # noqa: F811
    """Every point on the list of those that are measured in full, around the lengths from which two, four and eight waves of a
    workgroup have points of their own."""
    _same(both, *_data(kind, B, N, d, K, seed=N + d + K))
