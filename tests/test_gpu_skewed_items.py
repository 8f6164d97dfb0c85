"""Items of a cluster that holds far more points than the others (item_length in csrc/fk_update.hip): longer ones, which
still cover every point once, around the sizes where their number is cut."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,N,d,K", [
    (torch.float16, 40000, 32, 300), (torch.bfloat16, 30001, 100, 500), (torch.float32, 20000, 104, 660), (torch.float32, 9000, 512, 17),
    (torch.float16, 4194305, 8, 40), (torch.bfloat16, 70001, 264, 3),
])
@pytest.mark.parametrize("big", [2047, 2048, 2049, 4097, 8193, -1])
def test_items_of_a_large_cluster(dtype, N, d, K, big):
    g = torch.Generator(device=DEV).manual_seed(N + d)
    X = torch.randn((1, N, d), generator=g, device=DEV).to(dtype)
    C0 = torch.zeros((1, K, d), device=DEV)
    label = torch.randint(0, K, (1, N), generator=g, device=DEV, dtype=torch.int32)
    label[0, torch.randperm(N, generator=g, device=DEV)[: big if big > 0 else N - N // 8]] = K // 2
    try:
        fk.fk_set_option("fused_update", 0)
        fk.fk_set_option("gather_update", 0)
        C, _, n = fk.fk_update(X, label, C0)
    finally:
        fk.fk_set_option("fused_update", -1)
        fk.fk_set_option("gather_update", -1)
    at = label[0].long()
    assert torch.equal(n[0].long(), torch.bincount(at, minlength=K))
    x = X[0].double()
    order = torch.argsort(at, stable=True)
    ends = n[0].long().cumsum(0)

    def sums(v):                                  # by cluster, from a running sum in 64 bits
        run = torch.cat([torch.zeros((1, d), dtype=torch.float64, device=DEV), v[order].cumsum(0)])
        return run[ends] - run[ends - n[0].long()]

    total, size = sums(x), sums(x.abs())
    m = n[0].double().clamp(min=1)[:, None]
    # n additions of 2^-24 of the magnitudes' sum each at most, divided by n; the oracle's running sums: N 2^-53 of theirs
    bound = 2.0 ** -24 * (size + 1) + 2.0 ** -52 * N * size.sum(0) / m
    assert ((C[0].double() - total / m).abs() <= bound).all()


@pytest.mark.parametrize("dtype,N,d,K", [(torch.float32, 300000, 96, 400), (torch.float32, 100000, 256, 300), (torch.float16, 300000, 200, 700), (torch.bfloat16, 4194400, 64, 64)])
def test_no_long_chain_of_additions(dtype, N, d, K):
    """Every column holds one 1 and otherwise 2^-24, which an addition to the 1 loses whole: the sum is off by as many of
    them as follow the 1 in its chain.  Items of 160 to 512 rows (3075 for four waves) and their merge: no term passes through more than the 128
    additions of a wave that adds one item of 256 narrow rows, two at a time, row by row."""
    X = torch.full((1, N, d), 2.0 ** -24, dtype=dtype, device=DEV)
    X[0, torch.arange(d, device=DEV) * 997 % N, torch.arange(d, device=DEV)] = 1.0     # any place in a chain
    label = torch.full((1, N), K // 2, dtype=torch.int32, device=DEV)
    try:
        fk.fk_set_option("fused_update", 0)
        fk.fk_set_option("gather_update", 0)
        C, _, _ = fk.fk_update(X, label, torch.zeros((1, K, d), device=DEV))
    finally:
        fk.fk_set_option("fused_update", -1)
        fk.fk_set_option("gather_update", -1)
    total = 1 + (N - 1) * 2.0 ** -24
    # ... each good to 2^-24 of the whole, and the rounding of the mean
    assert (C[0, K // 2].double() * N - total).abs().max() <= (128 + 1) * 2.0 ** -24 * total
