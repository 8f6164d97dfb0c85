"""Out-of-core calls on both sides of the line between copies beside the kernels and copies read by a kernel on the caller's stream
(fk_lloyd_ooc in csrc/fk_ooc.hip): rows that start at 16, 4 and 2 bytes, one chunk and several, the in-core call's answers."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,N,d,K,chunk", [
    (torch.float16, 1, 8, 1, 1), (torch.bfloat16, 257, 9, 5, 100), (torch.float16, 5001, 33, 40, 1001), (torch.float16, 4000, 34, 17, 999),
    (torch.float32, 3001, 17, 30, 1000), (torch.float32, 20000, 100, 70, 20000), (torch.float16, 65536, 128, 40, 30001),   # 16 MiB
    (torch.float16, 65537, 128, 40, 30001), (torch.bfloat16, 100001, 101, 50, 33001), (torch.float32, 120000, 64, 33, 120000),
    (torch.float16, 2000, 5, 9, 700),
])
@pytest.mark.parametrize("iters", [1, 3])
def test_out_of_core_gives_the_in_core_answers(dtype, N, d, K, chunk, iters):
    g = torch.Generator().manual_seed(N + d)
    centre = 6 * torch.randn((K, d), generator=g)
    lab = torch.cat([torch.arange(min(K, N)), torch.randint(0, K, (max(0, N - K),), generator=g)])
    X = (centre[lab] + 0.2 * torch.randn((N, d), generator=g)).to(dtype)
    C0 = X[:K].float().to(DEV).contiguous()
    host = torch.empty((N + 8, d), dtype=dtype, pin_memory=True)[8:]      # not the start of its allocation
    host.copy_(X)
    before = host.clone()
    ws = torch.empty(fk.fk_ooc_workspace_bytes(chunk, d, K, dtype), dtype=torch.uint8, device=DEV)
    C, D = C0.clone(), C0[None].clone()
    a, n = fk.fk_lloyd_ooc(host, C, iters, dev_ws=ws, chunk_rows=chunk)
    b, m, _ = fk.fk_lloyd_iter(X[None].to(DEV).contiguous(), D, iters)
    assert torch.equal(a, b[0]) and torch.equal(n, m[0]) and torch.equal(host, before)
    # the same n terms in two orders: n 2^-23 of their largest each (additions in the matrix pipe included), divided by n
    assert ((C - D[0]).abs() <= 2 * 2.0 ** -23 * n.amax() * X.float().abs().max()).all()
    one = C0.clone()
    for _ in range(iters):
        c, _ = fk.fk_lloyd_ooc(host, one, 1, dev_ws=ws, chunk_rows=chunk)
    assert torch.equal(one, C) and torch.equal(c, a)
