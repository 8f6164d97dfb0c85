"""The update of small instances without a sort (gather_update_kernel in csrc/fk_update.hip): counts of the sorted path and
means of the 64-bit sums, over parts, waves per workgroup, widths, ids out of range and one cluster with everything."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,N,d,K", [
    (1, 1, 8, 1), (2, 63, 9, 3), (3, 255, 16, 5), (1, 257, 5, 40), (1, 1025, 33, 300), (2, 4097, 100, 70), (1, 5000, 255, 2),
    (1, 6001, 256, 17), (1, 3000, 260, 600), (1, 2500, 511, 33), (1, 2049, 512, 1), (5, 1111, 64, 200), (1, 16384, 24, 130),
])
def test_gathered_update(dtype, B, N, d, K):
    g = torch.Generator(device=DEV).manual_seed(N + d + K)
    X = torch.randn((B, N, d), generator=g, device=DEV).to(dtype)
    C0 = torch.randn((B, K, d), generator=g, device=DEV)
    skewed = (K * torch.rand((B, N), generator=g, device=DEV) ** 4).int() - 1      # -1 and K belong to the first and the last
    for label in (skewed, torch.full_like(skewed, K // 2), skewed + 2):
        at = label.clamp(0, K - 1).long()
        n = torch.stack([torch.bincount(a, minlength=K) for a in at])
        x = X.double().cpu()
        total = torch.zeros((B, K, d), dtype=torch.float64).scatter_add_(1, at.cpu()[..., None].expand(B, N, d), x).to(DEV)
        size = torch.zeros((B, K, d), dtype=torch.float64).scatter_add_(1, at.cpu()[..., None].expand(B, N, d), x.abs()).to(DEV)
        want = torch.where(n[..., None] > 0, total / n.clamp(min=1)[..., None], C0.double())
        # n additions of 2^-24 of the magnitudes' sum each at most, divided by n, and the rounded mean
        bound = 2.0 ** -24 * (size + want.abs())
        try:
            for parts in (-1, 1, 2, 7):
                fk.fk_set_option("fused_update", 0)
                fk.fk_set_option("gather_update", parts)
                assert parts < 0 or f"gather(parts={parts}," in fk.fk_plan(B, N, d, K, dtype)
                C, lp, m = fk.fk_update(X, label, C0)
                assert torch.equal(m.long(), n)
                assert ((C.double() - want).abs() <= bound).all()
                assert torch.equal(lp, C.to(dtype))
                again = fk.fk_update(X, label, C0)
                assert torch.equal(C, again[0]) and torch.equal(lp, again[1])
                if B == 1 and parts > 0:
                    # inside a fit: the next assignment reads the fragments and biases written here
                    D = C0.clone()
                    a, c, _ = fk.fk_lloyd_iter(X, D, 2)
                    fk.fk_set_option("gather_update", 0)
                    E = C0.clone()
                    b, e, _ = fk.fk_lloyd_iter(X, E, 1)
                    fk.fk_set_option("gather_update", parts)
                    F = C0.clone()
                    f, h, _ = fk.fk_lloyd_iter(X, F, 1)
                    assert torch.equal(b, f) and torch.equal(e, h)
                    h, _, _ = fk.fk_lloyd_iter(X, F, 1)
                    assert torch.equal(a, h) and torch.equal(D, F)
        finally:
            fk.fk_set_option("gather_update", -1)
            fk.fk_set_option("fused_update", -1)


@pytest.mark.parametrize("parts", [1, 3])
@pytest.mark.parametrize("dtype,N,d,K,chunk", [(torch.float16, 6001, 72, 50, 2001), (torch.bfloat16, 7100, 20, 33, 1024), (torch.float32, 4100, 3, 10, 1000)])
def test_out_of_core_chunks(dtype, N, d, K, chunk, parts):
    g = torch.Generator().manual_seed(N)
    centre = 8 * torch.randn((K, d), generator=g)
    lab = torch.cat([torch.arange(K), torch.randint(0, K, (N - K,), generator=g)])
    X = (centre[lab] + 0.3 * torch.randn((N, d), generator=g)).to(dtype).pin_memory()
    got = []
    try:
        for v in (0, parts):
            fk.fk_set_option("gather_update", v)
            ws = torch.empty(fk.fk_ooc_workspace_bytes(chunk, d, K, dtype), dtype=torch.uint8, device=DEV)
            C, D = (X[:K].float().to(DEV).contiguous() for _ in range(2))
            a, n = fk.fk_lloyd_ooc(X, C, 3, dev_ws=ws, chunk_rows=chunk)
            for _ in range(3):
                fk.fk_lloyd_ooc(X, D, 1, dev_ws=ws, chunk_rows=chunk)
            assert torch.equal(C, D)             # chunks that wait for their turn (merged) and those that do not
            got.append((a, n, C))
    finally:
        fk.fk_set_option("gather_update", -1)
    (a, n, C), (b, m, D) = got
    assert torch.equal(a, b) and torch.equal(n, m)
    # the same n terms in two orders: n 2^-24 of their largest each, divided by n
    assert ((C - D).abs() <= 2 * 2.0 ** -24 * n.amax() * X.float().abs().max()).all()


@pytest.mark.parametrize("parts", [1, 2])
def test_stage_timer_books_all_of_an_update_without_a_sort(parts):
    """The launch under the reduction, the merge of parts under the merge, and there too, with parts and without,
    what is enqueued between two updates: the re-layout of the centroids that the next call starts from."""
    g = torch.Generator(device=DEV).manual_seed(3)
    X = torch.randn((1, 3000, 128), generator=g, device=DEV).half()
    C = X[:, :300].float().contiguous()
    try:
        fk.fk_set_option("gather_update", parts)
        fk.fk_lloyd_iter(X, C, 1)
        fk.fk_stage_timer_start()
        for _ in range(2):
            fk.fk_lloyd_iter(X, C, 2)
        st = fk.fk_stage_timer_stop()
    finally:
        fk.fk_set_option("gather_update", -1)
    assert {k: n for k, (_, n) in st.items()} == {"assign": 4, "sort": 0, "reduce": 4, "finalize": 4 if parts > 1 else 0}
    assert st["assign"][0] > 0 and st["reduce"][0] > 0 and st["finalize"][0] > 0 and st["sort"][0] == 0


@pytest.mark.parametrize("dtype,N,d,K", [(torch.float32, 8000, 512, 100), (torch.bfloat16, 8192, 128, 1000), (torch.float16, 5000, 256, 300)])
def test_no_long_chain_of_additions(dtype, N, d, K):
    """Every column holds one 1 and otherwise 2^-24, which an addition to the 1 loses whole: the sum is off by as many of
    them as follow the 1 in its chain.  No term passes through more than 64 additions, in batches and on to the mean,
    with the sort (items of 32 rows, their merge) or without."""
    X = torch.full((1, N, d), 2.0 ** -24, dtype=dtype, device=DEV)
    X[0, torch.arange(d, device=DEV) * 997 % N, torch.arange(d, device=DEV)] = 1.0     # any place in a chain
    label = torch.full((1, N), K // 2, dtype=torch.int32, device=DEV)
    total = 1 + (N - 1) * 2.0 ** -24
    for parts in (-1, 0):
        try:
            fk.fk_set_option("gather_update", parts)
            assert ("gather" in fk.fk_plan(1, N, d, K, dtype)) == (parts != 0)
            C, _, _ = fk.fk_update(X, label, torch.zeros((1, K, d), device=DEV))
        finally:
            fk.fk_set_option("gather_update", -1)
        # ... each good to 2^-24 of the whole, and the rounding of the mean
        assert (C[0, K // 2].double() * N - total).abs().max() <= (64 + 1) * 2.0 ** -24 * total


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N,d,K,parts", [
    # four and eight waves; shares of one block of 256 keys a wave and around those from which waves add as they go;
    # lists around 256 rows; whole and broken batches of rows, of 64 and more rows to a load
    (256, 64, 3, 1), (257, 8, 3, 1), (513, 512, 5, 2), (1023, 100, 520, 1), (2048, 33, 600, 2), (4097, 256, 300, 1), (8191, 16, 300, 1), (8192, 40, 300, 1),
    (8449, 9, 270, 1), (16383, 128, 40, 1), (16384, 24, 40, 1), (16641, 320, 7, 1), (40000, 32, 9, 2), (70001, 8, 2, 3),
])
def test_every_row_counts_once(dtype, N, d, K, parts):
    """Small whole numbers: every partial sum is exact, so that a row lost or taken twice shows."""
    g = torch.Generator(device=DEV).manual_seed(N + d)
    X = torch.randint(-3, 4, (1, N, d), generator=g, device=DEV)
    X[..., 0] = 1 + torch.arange(N, device=DEV) % 3
    u = torch.rand((1, N), generator=g, device=DEV)
    C0 = torch.randn((1, K, d), generator=g, device=DEV)
    for label in ((K * u).int(), (K * u ** 4).int(), torch.full((1, N), K // 2, dtype=torch.int32, device=DEV), (K * (torch.arange(N, device=DEV)[None] // 64) // (N // 64 + 1)).int()):
        label = label.clamp(max=K - 1)
        total = torch.zeros((K, d), dtype=torch.int64).index_add_(0, label[0].long().cpu(), X[0].cpu())
        n = torch.bincount(label[0].cpu(), minlength=K)
        want = torch.where(n[:, None] > 0, (total.double() / n.clamp(min=1)[:, None]).float(), C0[0].cpu())
        try:
            fk.fk_set_option("fused_update", 0)
            fk.fk_set_option("gather_update", parts)
            C, _, m = fk.fk_update(X.to(dtype), label, C0)
        finally:
            fk.fk_set_option("gather_update", -1)
            fk.fk_set_option("fused_update", -1)
        assert torch.equal(m[0].cpu().long(), n) and torch.equal(C[0].cpu(), want)


@pytest.mark.parametrize("N,d,K,dtype", [(16384, 512, 64, torch.float32), (1024, 512, 20, torch.float32), (8192, 128, 1000, torch.bfloat16)])
def test_as_many_parts_as_the_workspace_has_room_for(N, d, K, dtype):
    g = torch.Generator(device=DEV).manual_seed(N)
    X = torch.randint(-3, 4, (1, N, d), generator=g, device=DEV).to(dtype)
    label = (K * torch.rand((1, N), generator=g, device=DEV) ** 4).int()
    C0 = torch.zeros((1, K, d), device=DEV)
    want = fk.fk_update(X, label, C0)
    try:
        fk.fk_set_option("gather_update", 0)
        room = fk.fk_workspace_bytes(1, N, d, K, dtype)
    finally:
        fk.fk_set_option("gather_update", -1)
    ws = torch.full((room + 4096,), 0x55, dtype=torch.uint8, device=DEV)
    got = fk.fk_update(X, label, C0, ws=ws[:room])
    assert all(torch.equal(a, b) for a, b in zip(got, want))                      # sums of small whole numbers are exact
    assert bool((ws[room:] == 0x55).all())


@pytest.mark.parametrize("B,N,d,K,parts", [
    # workgroups per instance odd, even, a multiple of four and of eight; more turns than clusters
    (41, 300, 8, 3, 1), (23, 270, 24, 10, 1), (70, 300, 16, 4, 1), (19, 513, 12, 8, 1), (9, 1000, 32, 12, 2), (33, 260, 8, 1, 8), (5, 700, 100, 24, 3), (300, 64, 8, 16, 1),
])
def test_every_cluster_of_every_instance_has_its_turn(B, N, d, K, parts):
    """Clusters change places among the workgroups from instance to instance.  Sums of small whole numbers are exact."""
    g = torch.Generator(device=DEV).manual_seed(B + N)
    X = torch.randint(-3, 4, (B, N, d), generator=g, device=DEV)
    label = (K * torch.rand((B, N), generator=g, device=DEV) ** 3).int()
    at = (label.long() + K * torch.arange(B, device=DEV)[:, None]).view(-1).cpu()
    total = torch.zeros((B * K, d), dtype=torch.int64).index_add_(0, at, X.view(-1, d).cpu())
    n = torch.bincount(at, minlength=B * K)
    C0 = torch.randn((B, K, d), generator=g, device=DEV)
    want = torch.where(n[:, None] > 0, (total.double() / n.clamp(min=1)[:, None]).float(), C0.view(-1, d).cpu())
    try:
        fk.fk_set_option("fused_update", 0)
        fk.fk_set_option("gather_update", parts)
        for dtype in (torch.float16, torch.float32):
            C, _, m = fk.fk_update(X.to(dtype), label, C0)
            assert torch.equal(m.view(-1).cpu().long(), n) and torch.equal(C.view(-1, d).cpu(), want)
    finally:
        fk.fk_set_option("gather_update", -1)
        fk.fk_set_option("fused_update", -1)
