"""GPU parity of the loads that go past the caches: the assembly on both sides of the size from which it uses them, and
the weight gradient with one tile and with several in each dimension of the result."""
import pytest
import torch

from paper_2409_14939_amd import binding as B
from test_gpu_update import run_case

pytestmark = pytest.mark.gpu
STREAM_BYTES = 160 << 20


@pytest.mark.parametrize("feat,dtype", [(257, torch.float32), (6, torch.float32), (131, torch.bfloat16)])
@pytest.mark.parametrize("more", [0, 1])
def test_assembly_around_the_size(feat, dtype, more):
    row = feat * (4 if dtype == torch.float32 else 2)
    n = (STREAM_BYTES - 1) // row + more                    # the last size below the line, the first on it
    assert (n * row >= STREAM_BYTES) == bool(more)
    g = torch.Generator(device="cuda")
    g.manual_seed(feat)
    prev = torch.empty((1000, feat), dtype=dtype, device="cuda").normal_(generator=g)
    load = torch.empty((777, feat), dtype=dtype, device="cuda").normal_(generator=g)
    src = torch.randint(-777, 1000, (n,), generator=g, device="cuda", dtype=torch.int32)
    out = B.fastgl_assemble_rows(prev, load, src, 777)
    assert torch.equal(out, torch.cat([load.flip(0), prev])[src.long() + 777])


@pytest.mark.parametrize("M,K,N", [(1500, 100, 100), (1501, 130, 99), (1501, 101, 130), (1500, 131, 131), (1500, 4, 100)])
@pytest.mark.parametrize("relu", [False, True])
def test_weight_gradient_by_number_of_tiles(M, K, N, relu):
    run_case(M, K, N, relu, bias=True, seed=M + K + N, what="tiles")


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("M", [204_600, 204_601])          # 100 + 64 columns: below 128 MB, from where one tile's operands go past the caches
def test_weight_gradient_around_the_size(M, relu):
    """Against float64; the bound of the parity tests: a chain as long as a slab, and the rounding of the result."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    H, dY, Y = (torch.empty((M, n), device="cuda").normal_(generator=g) for n in (100, 64, 64))
    _, dW, db = B.fastgl_update_bwd(H, torch.ones((100, 64), device="cuda"), Y if relu else None, dY, relu, want=("dW", "db"))
    dZ = (dY * (Y > 0) if relu else dY).double()
    ref, size = H.double().T @ dZ, H.double().abs().T @ dZ.abs()
    u = (min(M, B.fastgl_update_slab_rows(M, 100, 64)) + 4) * 2.0 ** -24
    assert bool(((dW.double() - ref).abs() <= u * size + 2.0 ** -24 * ref.abs()).all())
    assert bool(((db.double() - dZ.sum(0)).abs() <= u * dZ.abs().sum(0)).all())
