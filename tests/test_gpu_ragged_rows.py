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
    for fused, gather in ((-1, -1), (0, -1), (0, 0)):
        try:
            fk.fk_set_option("fused_update", fused)
            fk.fk_set_option("gather_update", gather)
            assert gather < 0 or "sort=" in fk.fk_plan(B, N, d, K, dtype)
            p, q = fk.fk_update(X, lab, C), fk.fk_update(Xp, lab, Cp)
            c, cp = C.clone(), Cp.clone()
            u, v = fk.fk_lloyd_iter(X, c, 3), fk.fk_lloyd_iter(Xp, cp, 3)
        finally:
            fk.fk_set_option("fused_update", -1)
            fk.fk_set_option("gather_update", -1)
        assert torch.equal(p[0], q[0][..., :d]) and torch.equal(p[1], q[1][..., :d]) and torch.equal(p[2], q[2])
        assert torch.equal(u[0], v[0]) and torch.equal(u[1], v[1]) and torch.equal(c, cp[..., :d]) and torch.equal(u[2], v[2][..., :d])


@pytest.mark.parametrize("N", [500, 9000, 140000])
@pytest.mark.parametrize("d", [130, 160, 180, 192, 210, 224, 250, 300, 320, 370, 400])
def test_every_compiled_width_equals_zero_padded_rows(d, N):
    """Rows between 128 and 512 features take kernels for 10, 12, 14, 16, 20, 24 or 32 chunks of 16: the chunks
    that a wider kernel multiplies on top are zeros and change no bit."""
    g = torch.Generator().manual_seed(N + d)
    X, C = (3 * torch.randn((1, n, d), generator=g).half().to(DEV) for n in (N, 400))
    wide = [F.pad(t, (0, 512 - d)) for t in (X, C)]
    for u, v in zip(fk.fk_assign(X, C, min_dist=True), fk.fk_assign(*wide, min_dist=True)):
        assert torch.equal(u, v)
    c, cw = X[:, :400].float().contiguous(), wide[0][:, :400].float().contiguous()
    u, v = fk.fk_lloyd_iter(X, c, 1), fk.fk_lloyd_iter(wide[0], cw, 1)
    assert torch.equal(u[0], v[0]) and torch.equal(u[1], v[1])
    # how a wave splits a segment's rows depends on the row width: the same n terms in two orders, each
    # good to n 2^-24 of their largest
    assert ((c - cw[..., :d]).abs() <= 2 * u[1].amax() * 2.0 ** -24 * X.abs().amax().float()).all()
