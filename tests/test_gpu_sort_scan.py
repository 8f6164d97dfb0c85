"""The counting sort with and without its scan kernel (sort_scatter_scans in csrc/fk_common.h): around the numbers of
workgroups, bins and instances where the one takes over from the other, against a stable sort."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TILE = 4096


@pytest.mark.parametrize("B,blocks,K", [
    (1, 1, 7), (1, 2, 1), (1, 2, 1024), (1, 31, 1000), (1, 33, 1000), (1, 64, 64), (1, 65, 64), (3, 48, 33), (1, 64, 512), (1, 65, 512),
    (20, 48, 300), (20, 49, 300), (22, 48, 16), (45, 24, 16), (45, 25, 16), (1, 5, 4096), (1, 70, 4096), (300, 2, 3),
])
@pytest.mark.parametrize("tail", [0, 1, 4095])
def test_sort_equals_a_stable_sort(B, blocks, K, tail):
    N = blocks * TILE - tail
    g = torch.Generator(device=DEV).manual_seed(N + K)
    a = torch.randint(0, max(1, K - 1), (B, N), generator=g, device=DEV, dtype=torch.int32)      # the last stays empty
    idx, off = fk.fk_sort_inverse(a, K)
    want = torch.sort(a, dim=1, stable=True)
    assert torch.equal(idx, want.indices.int())
    edges = torch.arange(K + 1, device=DEV, dtype=torch.int32).expand(B, K + 1).contiguous()
    assert torch.equal(off, torch.searchsorted(want.values, edges, out_int32=True))
