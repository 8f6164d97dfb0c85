"""Out-of-core iterations that go through the chunks back and forth: one call equals single-iteration calls
(which always go forward) up to the order of the fp32 sums, for every number of chunks and a short last one."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,N,d,K,chunk", [
    (torch.float16, 5000, 64, 20, 5000), (torch.float16, 5001, 100, 20, 2600), (torch.bfloat16, 9001, 33, 300, 2048),
    (torch.float32, 7000, 40, 30, 1500), (torch.float32, 4100, 3, 10, 1000),
])
def test_back_and_forth_equals_single_iterations(dtype, N, d, K, chunk):
    g = torch.Generator().manual_seed(N + d)
    centre = 8 * torch.randn((K, d), generator=g)
    lab = torch.cat([torch.arange(K), torch.randint(0, K, (N - K,), generator=g)])
    X = (centre[lab] + 0.3 * torch.randn((N, d), generator=g)).to(dtype).pin_memory()
    ws = torch.empty(fk.fk_ooc_workspace_bytes(chunk, d, K, dtype), dtype=torch.uint8, device=DEV)
    C, D = (X[:K].float().to(DEV).contiguous() for _ in range(2))
    a, n = fk.fk_lloyd_ooc(X, C, 4, dev_ws=ws, chunk_rows=chunk)
    for _ in range(4):
        b, m = fk.fk_lloyd_ooc(X, D, 1, dev_ws=ws, chunk_rows=chunk)
    assert torch.equal(a, b) and torch.equal(n, m)
    # sums of N / K terms and a handful of chunks in two orders, in fp32
    assert ((C - D).abs() <= 64 * 2.0 ** -24 * C.abs().amax()).all()
