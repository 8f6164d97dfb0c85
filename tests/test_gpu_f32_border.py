"""Points almost in the middle between two centroids: the filtered and the direct fp32 assignment round the same sums in the same
order, so that they agree on these too."""
import pytest

from tests.test_gpu_f32_filter import _data, both  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 48, 60, 64, 128, 256])
@pytest.mark.parametrize("seed", [0, 1000, 2000])
def test_points_between_two_centroids(both, d, seed):  # noqa: F811
    X, C = _data("border", 2, 4095, d, 97, seed=4095 + d + 97 + seed)
    (a1, _), (a0, _) = both(X, C)
    assert (a1 == a0).all()
