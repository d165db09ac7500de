"""What the Python calls accept, refuse and raise (argument marshalling, not results)."""
import ctypes
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import blockgen as bg
from gpu_util import dev_i32
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


def small_blocks():
    rng = np.random.default_rng(4)
    out = []
    for nd, ns in ((20, 50), (7, 30)):
        b = bg.random_block(rng, nd, ns, 4.0)
        out.append((dev_i32(b.indptr), dev_i32(b.indices), b.num_src))
    return out


def test_blocks_are_a_sequence():
    """A generator cannot be gone through twice: refused before anything is built, like sets and dicts."""
    blocks = small_blocks()
    for bad in ((b for b in blocks), iter(blocks), set(blocks), dict.fromkeys(blocks), 3, [(x for x in blocks[0])]):
        with pytest.raises(TypeError):
            B.fastgl_block_plan_create_many(bad)
    with pytest.raises(ValueError):
        B.fastgl_block_plan_create_many([blocks[0][:2]])
    assert B.fastgl_block_plan_create_many([]) == []
    for good in (blocks, tuple(blocks), [list(b) for b in blocks]):
        assert [p.num_src for p in B.fastgl_block_plan_create_many(good)] == [50, 30]


def test_plan_memory_is_anything_indexed_by_block():
    blocks = small_blocks()
    need = max(B.fastgl_block_plan_bytes(ip.numel() - 1, ns, ix.numel()) for ip, ix, ns in blocks)
    need = -(-need // 256) * 256
    rows = torch.empty((2, need), dtype=torch.uint8, device="cuda")
    for mems in ([rows[0], rows[1]], {0: rows[0], 1: rows[1]}, rows, [rows[0], rows[1], None]):
        made = B.fastgl_block_plan_create_many(blocks, plan_mems=mems)
        assert [p.mem.data_ptr() for p in made] == [rows[0].data_ptr(), rows[1].data_ptr()]
    with pytest.raises(IndexError):
        B.fastgl_block_plan_create_many(blocks, plan_mems=[rows[0]])


@pytest.mark.parametrize("bad", [2.0, 2.7, "2", None, np.int64(2), np.float32(2)])
def test_sizes_are_ints(bad):
    """What the C types refuse is refused: nothing is truncated or parsed on the way."""
    ip, ix, ns = small_blocks()[0]
    X = torch.ones((ns, 4), device="cuda")
    rows = torch.zeros(2, dtype=torch.int32, device="cuda")
    for call in (lambda: B.fastgl_block_plan_create(ip, ix, bad), lambda: B.fastgl_block_plan_create(ip, ix, ns, bad),
                 lambda: B.fastgl_block_aggregate_fwd(ip, ix, None, bad, "sum", X),
                 lambda: B.fastgl_edge_weight_grad(ip, ix, bad, "sum", X, X[:20]),
                 lambda: B.fastgl_assemble_rows(X, X, rows, bad)):
        with pytest.raises(TypeError):
            call()
    assert B.fastgl_assemble_rows(X, X, rows, 2).shape == (2, 4)


def test_numbers_that_are_converted():
    """Offsets go through int(), the slope through float(): whatever those take."""
    gid = torch.arange(6, dtype=torch.int64, device="cuda")
    ref = B.fastgl_overlap_counts(gid, [0, 3, 6])[0]
    for offsets in (np.array([0, 3, 6]), [0, "3", 6.0], torch.tensor([0, 3, 6])):
        assert torch.equal(B.fastgl_overlap_counts(gid, offsets)[0], ref)
    ip, ix, ns = small_blocks()[0]
    el, er = torch.ones(20, device="cuda") * -1, torch.zeros(ns, device="cuda")
    for slope in ("0.25", np.float64(0.25), torch.tensor(0.25)):
        assert torch.equal(B.fastgl_edge_score_fwd(ip, ix, el, er, slope), B.fastgl_edge_score_fwd(ip, ix, el, er, 0.25))


def test_plan_is_an_ordinary_object():
    """Attributes may be added and the handle handed on: to another Plan, or to any object that carries it."""
    ip, ix, ns = small_blocks()[0]
    X = torch.randn((ns, 4), device="cuda")
    plan = B.fastgl_block_plan_create(ip, ix, ns)
    assert isinstance(plan.handle, ctypes.c_void_p)
    plan.epoch = 3
    ref = B.fastgl_block_aggregate_fwd(ip, ix, None, ns, "gcn", X, plan=plan)
    owner = B.Plan(plan.handle, plan.mem, ip, ix, ns)
    plan.handle = None
    plan.destroy()                                            # nothing left to destroy
    for p in (owner, SimpleNamespace(handle=owner.handle), SimpleNamespace(handle=owner.handle.value)):
        assert torch.equal(B.fastgl_block_aggregate_fwd(ip, ix, None, ns, "gcn", X, plan=p), ref)
    assert owner.export().din
    owner.destroy()
    assert owner.handle is None
    assert torch.equal(B.fastgl_block_aggregate_fwd(ip, ix, None, ns, "gcn", X, plan=owner), ref)   # as without a plan


def test_want_is_not_asked_for_results_that_are_passed_in():
    H, W, dY = (torch.randn(s, device="cuda") for s in ((5, 3), (3, 2), (5, 2)))
    ref = B.fastgl_update_bwd(H, W, None, dY, False)
    out = [torch.empty_like(t) for t in ref]
    got = B.fastgl_update_bwd(H, W, None, dY, False, None, *out)
    assert all(torch.equal(a, b) and a is c for a, b, c in zip(got, ref, out))
    ip, ix, ns = small_blocks()[0]
    plan = B.fastgl_block_plan_create(ip, ix, ns, B.PLAN_ALL | B.PLAN_PERM)
    el, er, g = torch.randn(20, device="cuda"), torch.randn(ns, device="cuda"), torch.randn(ix.numel(), device="cuda")
    ref = B.fastgl_edge_score_bwd(ip, ix, el, er, 0.2, g, plan)
    got = B.fastgl_edge_score_bwd(ip, ix, el, er, 0.2, g, plan, None, torch.empty_like(el), torch.empty_like(er))
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


def test_feature_matrices_with_further_dimensions_of_one():
    ip, ix, ns = small_blocks()[0]
    X, W = torch.randn((ns, 4), device="cuda"), torch.randn((4, 3), device="cuda")
    ids = torch.arange(5, device="cuda")
    ref = B.fastgl_block_aggregate_fwd(ip, ix, None, ns, "gcn", X)
    assert torch.equal(B.fastgl_block_aggregate_fwd(ip, ix, None, ns, "gcn", X[..., None]), ref)
    assert torch.equal(B.fastgl_gather_rows(X[..., None, None], ids), X[:5])
    assert torch.equal(B.fastgl_update_fwd(ref, W[..., None], None, False), B.fastgl_update_fwd(ref, W, None, False))
    for call in (lambda: B.fastgl_block_aggregate_fwd(ip, ix, None, ns, "gcn", X.view(ns, 2, 2)),
                 lambda: B.fastgl_gather_rows(X.view(-1), ids), lambda: B.fastgl_update_fwd(ref[..., None], W, None, False)):
        with pytest.raises(ValueError):
            call()
