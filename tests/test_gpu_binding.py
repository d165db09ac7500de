"""What the Python calls accept, refuse and raise (argument marshalling, not results)."""
import pytest
import torch

from paper_2409_14939_amd import binding as B

pytestmark = pytest.mark.gpu


def test_an_allocation_that_does_not_fit_raises_torchs_error():
    """The allocator's own limit refuses the request on the host; a smaller batch then goes through."""
    table = torch.ones((4, 1 << 14), device="cuda")
    ids = torch.zeros(1 << 20, dtype=torch.int64, device="cuda")
    torch.cuda.set_per_process_memory_fraction(0.02)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            B.fastgl_gather_rows(table, ids)                       # 64 GiB
        assert B.fastgl_gather_rows(table, ids[:8]).shape == (8, 1 << 14)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
