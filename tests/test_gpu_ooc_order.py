"""Out-of-core iterations that start with the chunks still in the buffers: one call gives the bits of
single-iteration calls (which always go forward), for every number of chunks and a short last one."""
import pytest
import torch

from paper_2603_09229_amd import binding as fk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,N,d,K,chunk", [
    (torch.float16, 5000, 64, 20, 5000), (torch.float16, 5001, 100, 20, 2600), (torch.bfloat16, 9001, 33, 300, 2048),
    (torch.float32, 7000, 40, 30, 1500), (torch.float32, 4100, 3, 10, 1000), (torch.float16, 6001, 72, 50, 2001),
    (torch.float16, 8192, 128, 40, 1024), (torch.bfloat16, 7100, 20, 33, 1024), (torch.float32, 9000, 64, 25, 1000),
])
@pytest.mark.parametrize("room", [True, False])
@pytest.mark.parametrize("gather", [-1, 0])
def test_one_call_gives_the_bits_of_single_iterations(dtype, N, d, K, chunk, room, gather):
    g = torch.Generator().manual_seed(N + d)
    centre = 8 * torch.randn((K, d), generator=g)
    lab = torch.cat([torch.arange(K), torch.randint(0, K, (N - K,), generator=g)])
    X = (centre[lab] + 0.3 * torch.randn((N, d), generator=g)).to(dtype).pin_memory()
    # (without the room for the sums of chunks taken early every iteration goes forward)
    need = fk.fk_ooc_workspace_bytes(chunk, d, K, dtype) - (0 if room else 256)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    C, D = (X[:K].float().to(DEV).contiguous() for _ in range(2))
    try:
        fk.fk_set_option("gather_update", gather)          # (out of core that changes no size)
        a, n = fk.fk_lloyd_ooc(X, C, 4, dev_ws=ws, chunk_rows=chunk)
        for _ in range(4):
            b, m = fk.fk_lloyd_ooc(X, D, 1, dev_ws=ws, chunk_rows=chunk)
    finally:
        fk.fk_set_option("gather_update", -1)
    assert torch.equal(a, b) and torch.equal(n, m) and torch.equal(C, D)
