"""Row widths that are no multiple of 8: the kernels read and write the caller's rows as they are stored
and must give the bits that rows padded with zeros to the next multiple of 8 give."""
import pytest
import torch
import torch.nn.functional as F

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # one per kernel that reads rows, widths with every remainder, K with empty clusters and ragged tiles
    (torch.float16, 1, 3001, 9, 40), (torch.float16, 1, 5003, 100, 300), (torch.bfloat16, 2, 1501, 63, 1100),
    (torch.bfloat16, 3, 2049, 101, 70), (torch.float16, 1, 70001, 30, 290), (torch.bfloat16, 1, 4099, 130, 33),
    (torch.float16, 1, 20011, 300, 65), (torch.float16, 1, 9001, 511, 260), (torch.bfloat16, 1, 3000, 12, 16),
    (torch.float16, 2, 777, 125, 5), (torch.float16, 1, 900, 3, 40), (torch.bfloat16, 1, 263000, 67, 70),
    (torch.float32, 1, 3001, 9, 40), (torch.float32, 2, 2003, 70, 65), (torch.float32, 1, 5003, 101, 500),
    (torch.float32, 1, 270001, 33, 20), (torch.float32, 1, 1500, 205, 12), (torch.float32, 1, 70001, 131, 16),
    (torch.float32, 1, 1201, 510, 70), (torch.float32, 1, 3000, 7, 100),
]


@pytest.mark.parametrize("dtype,B,N,d,K", CASES)
def test_ragged_rows_equal_zero_padded_rows(dtype, B, N, d, K):
    g = torch.Generator().manual_seed(N + d + K)
    pad = -d % 8
    X = (3 * torch.randn((B, N, d), generator=g)).to(dtype).to(DEV)
    C = (3 * torch.randn((B, K, d), generator=g)).to(dtype).float().to(DEV)
    lab = torch.randint(0, max(1, K - 2), (B, N), generator=g, dtype=torch.int32).to(DEV)    # the last two stay empty
    Xp, Cp = F.pad(X, (0, pad)), F.pad(C, (0, pad))
    for u, v in zip(fk.fk_assign(X, C.to(dtype), min_dist=True), fk.fk_assign(Xp, Cp.to(dtype), min_dist=True)):
        assert torch.equal(u, v)
    u, v = fk.fk_update(X, lab, C), fk.fk_update(Xp, lab, Cp)
    assert torch.equal(u[0], v[0][..., :d]) and torch.equal(u[1], v[1][..., :d]) and torch.equal(u[2], v[2])
    for fused in (-1, 0):
        try:
            fk.fk_set_option("fused_update", fused)
            c, cp = C.clone(), Cp.clone()
            u, v = fk.fk_lloyd_iter(X, c, 3), fk.fk_lloyd_iter(Xp, cp, 3)
        finally:
            fk.fk_set_option("fused_update", -1)
        assert torch.equal(u[0], v[0]) and torch.equal(u[1], v[1]) and torch.equal(c, cp[..., :d]) and torch.equal(u[2], v[2][..., :d])
