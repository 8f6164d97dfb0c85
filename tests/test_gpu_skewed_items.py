"""Items of a cluster that holds far more points than the others (item_length in csrc/fk_update.hip): longer ones, which
still cover every point once, around the sizes where their number is cut."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,N,d,K,R,balance", [
    # rows per item and the balance of item_length, which give the sizes where items get longer
    (torch.float16, 40000, 32, 300, 32, 2.0), (torch.bfloat16, 30001, 100, 500, 32, 0.5), (torch.float32, 20000, 104, 660, 32, 1.0),
    (torch.float32, 9000, 512, 17, 32, 4.0), (torch.float16, 4194305, 8, 40, 1025, 2.0), (torch.bfloat16, 60001, 264, 300, 32, 2.0),
])
def test_items_of_a_large_cluster(dtype, N, d, K, R, balance):
    """Small whole numbers: every partial sum is exact, so that a row lost or taken twice shows."""
    try:
        fk.fk_set_option("fused_update", 0)
        fk.fk_set_option("gather_update", 0)
        assert f"(rows_per_item={R})" in fk.fk_plan(1, N, d, K, dtype)
        g = torch.Generator(device=DEV).manual_seed(N + d)
        X = torch.randint(-3, 4, (1, N, d), generator=g, device=DEV, dtype=torch.int8)
        X[0, :, 0] = (1 + torch.arange(N, device=DEV) % 3).to(torch.int8)
        x = X.to(dtype)
        C0 = torch.zeros((1, K, d), device=DEV)
        # sizes at both sides of one more item than `most` allows, of the next length, and around whole items
        most = lambda n: max(64, int((balance * n) ** 0.5))
        grows = [n for n in range(R, N, R) if (n + R) // R > most(n + 1) and n // R <= most(n)]
        big = {1, R, N // 7, N - N // 8, N} | {n + e for n in grows[:2] + grows[-1:] for e in (0, 1, R + 1)} | {2 * n + 1 for n in grows[:1]}
        assert grows
        for n_big in sorted(n for n in big if 0 < n <= N):
            label = torch.randint(0, K - 1, (1, N), generator=g, device=DEV, dtype=torch.int32)
            label[label >= K // 2] += 1                                           # nobody else in the large cluster
            label[0, torch.randperm(N, generator=g, device=DEV)[:n_big]] = K // 2
            C, _, n = fk.fk_update(x, label, C0)
            at = label[0].long()
            assert int(n[0, K // 2]) == n_big and torch.equal(n[0].long(), torch.bincount(at, minlength=K))
            total = torch.zeros((K, d), dtype=torch.int32, device=DEV).index_add_(0, at, X[0].int()).double()
            assert torch.equal(C[0], (total / n[0].double().clamp(min=1)[:, None]).float())
    finally:
        fk.fk_set_option("fused_update", -1)
        fk.fk_set_option("gather_update", -1)


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
