"""GPU parity of the update phase with few result columns (its own kernels up to 8 columns), at the edges of
their lane groups: K around the lanes of a group and beyond one column block of dW, rows around the rows in
flight and beyond one slab, quads and single elements, both data types."""
import pytest
import torch

from paper_2409_14939_amd import binding as B
from test_gpu_update import run_case, test_update_parity_bf16 as bf16_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (3, 4, 2), (4, 3, 3), (5, 64, 1), (63, 255, 5), (65, 256, 8), (66, 260, 7),
                                   (129, 1030, 4), (70001, 20, 1), (70001, 7, 6), (1025, 100, 9),
                                   (20001, 64, 1), (20000, 65, 3), (20001, 3, 8), (20001, 130, 6)])
def test_narrow_update_parity(M, K, N):
    run_case(M, K, N, relu=M % 2 == 0, bias=M % 4 != 1, seed=M + K + N, what="narrow update")


@pytest.mark.parametrize("M,K,N", [(1500, 64, 1), (300, 18, 7), (257, 260, 8)])
def test_narrow_update_parity_bf16(M, K, N):
    bf16_case(M, K, N, M % 2 == 0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,K,N", [(5000, 64, 1), (5001, 30, 3), (3001, 300, 8), (3000, 64, 9), (3000, 64, 47), (2000, 100, 256)])
def test_results_do_not_depend_on_what_else_is_asked_for(M, K, N, dtype):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    H, W, dY = (torch.randn(s, generator=g, device="cuda").to(dtype) for s in ((M, K), (K, N), (M, N)))
    Y = B.fastgl_update_fwd(H, W, None, True)
    full = B.fastgl_update_bwd(H, W, Y, dY, True)
    for i, name in enumerate(("dH", "dW", "db")):
        assert torch.equal(B.fastgl_update_bwd(H, W, Y, dY, True, want=(name,))[i], full[i]), name


@pytest.mark.parametrize("M,K,N", [(5001, 30, 3), (3000, 64, 9), (3001, 300, 130), (2000, 100, 256)])
def test_db_alone_needs_neither_h_nor_w(M, K, N):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    H, W, dY = (torch.randn(s, generator=g, device="cuda") for s in ((M, K), (K, N), (M, N)))
    Y = B.fastgl_update_fwd(H, W, None, True)
    ref = B.fastgl_update_bwd(H, W, Y, dY, True, want=("db",))[2]
    db = torch.empty_like(ref)
    ws = torch.empty(B.fastgl_update_bwd_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda")
    B._check(B.lib().fastgl_update_bwd(None, None, B._ptr(Y), B._ptr(dY), M, K, N, 1, None, None, B._ptr(db), B._ptr(ws),
                                       ws.numel(), B._stream()))
    assert torch.equal(db, ref)
