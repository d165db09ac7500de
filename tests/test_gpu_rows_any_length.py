"""Feature rows of any length and alignment (the last 16-byte piece of a row ends with it and starts inside the piece
before) and rows shared by the lane groups of a wavefront: aggregation both ways, table gather, assembly and edge weight
gradient.  Against the oracle with the tolerances of the parity tests; copies byte for byte, with a guard around them."""
import numpy as np
import pytest
import torch

import blockgen as bg
import oracle
from paper_2409_14939_amd import binding as B
from gpu_util import assert_close, dev_feat, dev_i32, host_feat, make_inputs, read_i32
from test_gpu_parity import check_block

pytestmark = pytest.mark.gpu
FEATS = {"f32": [1, 2, 3, 4, 5, 7, 13, 17, 31, 63, 65, 101, 131, 255, 257, 602],
         "bf16": [1, 2, 3, 5, 7, 8, 9, 15, 17, 62, 99, 127, 129, 255, 257, 513, 530]}


def block_of(lengths, num_src, seed):
    rng = np.random.default_rng(seed)
    indptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return bg.Block(indptr, rng.integers(0, num_src, indptr[-1]).astype(np.int32), len(lengths), num_src)


@pytest.mark.parametrize("dtype,feat", [(d, f) for d in FEATS for f in FEATS[d]])
def test_widths(dtype, feat):
    blk = bg.random_block(np.random.default_rng(feat), 150, 333, 5.0, empty_frac=0.2, hub_rows=3, hub_deg=300)
    check_block(blk, "gcn", dtype, feat, feat % 2 == 0, True, feat, "odd width")


# runs of edges that end inside, at and between rows; rows over several groups; windows of more than 64 rows; none at all
SHAPES = {"one row": [200], "one edge": [1], "two edges": [0, 2, 0], "ends alone": [90] + [0] * 200 + [90],
          "empty among full": [0, 17] * 80, "256 each": [256] * 9, "one long in the middle": [1] * 70 + [257] + [1] * 70,
          "growing": list(range(120)), "mixed": [3, 0, 0, 250, 1, 1, 1, 0, 64, 63, 65, 0] * 7, "ones": [1] * 1000}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype,feat", [("f32", 4), ("f32", 30), ("f32", 64), ("f32", 128), ("f32", 256), ("bf16", 8),
                                        ("bf16", 100), ("bf16", 256)])
def test_row_shapes(shape, dtype, feat):
    blk = block_of(SHAPES[shape], 97, len(shape))
    check_block(blk, "mean", dtype, feat, False, True, feat, shape)
    check_block(blk, "gcn", dtype, feat, True, True, feat, shape + ", weighted")


def shifted(a, dtype, by):
    """`a` on the device at an address `by` elements past an aligned one."""
    t = dev_feat(a, dtype)
    room = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")
    room[by:] = t.reshape(-1)
    return room[by:].reshape(t.shape)


@pytest.mark.parametrize("dtype,feat,by", [("f32", 8, 1), ("f32", 129, 3), ("bf16", 64, 1), ("bf16", 33, 5)])
def test_any_alignment(dtype, feat, by):
    blk = bg.random_block(np.random.default_rng(by), 200, 411, 6.0, hub_rows=2, hub_deg=400)
    rng = np.random.default_rng(feat)
    X, G = make_inputs(rng, blk.num_src, feat, dtype), make_inputs(rng, blk.num_dst, feat, dtype)
    ip, ix, src = dev_i32(blk.indptr), dev_i32(blk.indices), blk.num_src
    Xd, Gd = shifted(X, dtype, by), shifted(G, dtype, by)
    out, dX = shifted(G, dtype, by), shifted(X, dtype, by)
    B.fastgl_block_aggregate_fwd(ip, ix, None, src, "sum", Xd, out=out)
    B.fastgl_block_aggregate_bwd(ip, ix, None, src, "sum", Gd, grad_X=dX)
    assert_close(host_feat(out, dtype), oracle.aggregate_fwd(blk.indptr, blk.indices, None, src, "sum", dtype, X), dtype)
    assert_close(host_feat(dX, dtype), oracle.aggregate_bwd(blk.indptr, blk.indices, None, src, "sum", dtype, G), dtype)
    dw = B.fastgl_edge_weight_grad(ip, ix, src, "sum", Xd, Gd)
    same = B.fastgl_edge_weight_grad(ip, ix, src, "sum", Xd.clone(), Gd.clone())
    assert torch.equal(dw, same)


@pytest.mark.parametrize("dtype,feat", [(d, f) for d in FEATS for f in FEATS[d]])
@pytest.mark.parametrize("by", [0, 1])
def test_copies(dtype, feat, by):
    rng = np.random.default_rng(feat)
    table = shifted(make_inputs(rng, 300, feat, dtype), dtype, by)
    load = shifted(make_inputs(rng, 50, feat, dtype), dtype, by)
    ids = torch.from_numpy(rng.integers(0, 300, 77)).cuda()
    bits = torch.int32 if dtype == "f32" else torch.int16

    def guarded():
        room = torch.full((77 * feat + 2 * 64 + by,), 7, dtype=bits, device="cuda")
        return room, room[64 + by:64 + by + 77 * feat].view(table.dtype).reshape(77, feat)

    room, out = guarded()
    B.fastgl_gather_rows(table, ids, out=out)
    assert torch.equal(out.view(bits), table.view(bits)[ids])
    assert (room[:64 + by] == 7).all() and (room[-64:] == 7).all()
    src = torch.from_numpy(rng.integers(-50, 300, 77).astype(np.int32)).cuda()
    room, out = guarded()
    B.fastgl_assemble_rows(table, load, src, 50, out=out)
    want = torch.where((src >= 0)[:, None], table.view(bits)[src.clamp(min=0).long()], load.view(bits)[(-1 - src).clamp(min=0).long()])
    assert torch.equal(out.view(bits), want)
    assert (room[:64 + by] == 7).all() and (room[-64:] == 7).all()


def check_edge_weight_grad(dtype, feat, edges_per_row, on_device):
    blk = bg.random_block(np.random.default_rng(feat), 140, 300, edges_per_row, empty_frac=0.2)
    rng = np.random.default_rng(feat)
    X, G = make_inputs(rng, blk.num_src, feat, dtype), make_inputs(rng, blk.num_dst, feat, dtype)
    x, g = (a.astype(np.float64) if dtype == "f32" else bg.bf16_bits_to_f32(a).astype(np.float64) for a in (X, G))
    got = B.fastgl_edge_weight_grad(dev_i32(blk.indptr), dev_i32(blk.indices), blk.num_src, "sum", on_device(X, dtype),
                                    on_device(G, dtype)).cpu().numpy()
    rows = np.repeat(np.arange(blk.num_dst), np.diff(blk.indptr))
    terms = np.abs(g[rows] * x[blk.indices]).sum(1)
    want = (g[rows] * x[blk.indices]).sum(1)
    # fp64 sums rounded once; bf16: products exact, a chain of at most feat fp32 additions
    bound = 2.0 ** -24 * np.abs(want) + (feat + 2) * (2.0 ** -52 if dtype == "f32" else 2.0 ** -24) * terms
    assert (np.abs(got - want) <= bound).all()


@pytest.mark.parametrize("dtype,feat", [(d, f) for d in FEATS for f in FEATS[d]])
@pytest.mark.parametrize("edges_per_row", [2.0, 300.0])
def test_edge_weight_grad(dtype, feat, edges_per_row):
    check_edge_weight_grad(dtype, feat, edges_per_row, dev_feat)


# rows of up to two pieces of every size, whole and ragged, at every address in a dword and just past aligned ones
@pytest.mark.parametrize("dtype,feat", [("f32", f) for f in range(1, 9)] + [("bf16", f) for f in range(1, 17)])
def test_edge_weight_grad_of_narrow_rows(dtype, feat):
    for by in (0, 1, 3):
        check_edge_weight_grad(dtype, feat, 7.0, lambda a, t: shifted(a, t, by))


def column_tiles(blk, feat, dtype):
    return B.lib().fastgl_aggregate_column_tiles(blk.num_dst, blk.num_src, blk.num_edges, feat, B.DTYPES[dtype])


@pytest.mark.parametrize("dtype,feat,weighted", [("f32", 256, True), ("f32", 384, False), ("bf16", 1280, True)])
def test_column_tiles_one_after_the_other(dtype, feat, weighted):
    """Wide rows read five times each out of a table of 128 MB and more: by column tiles, against the oracle; the same bits
    from an address at which the tiles of a row go together; rows of none, of a few, of the longest unchunked and of
    chunked length."""
    num_src = (128 << 20) // (feat * (4 if dtype == "f32" else 2)) + 1
    rng = np.random.default_rng(feat)
    lengths = np.concatenate([[0, 1, 256, 257, 3000], rng.integers(0, 60, 5 * num_src // 29)])
    blk = block_of(rng.permutation(lengths), num_src, feat)
    assert column_tiles(blk, feat, dtype) == feat * (4 if dtype == "f32" else 2) // 512
    X = make_inputs(rng, num_src, feat, dtype)
    w = rng.standard_normal(blk.num_edges).astype(np.float32) if weighted else None
    wd = None if w is None else torch.from_numpy(w).cuda()
    ip, ix = dev_i32(blk.indptr), dev_i32(blk.indices)
    aligned, moved = dev_feat(X, dtype), shifted(X, dtype, 2)
    assert aligned.data_ptr() % 128 == 0 and moved.data_ptr() % 128 != 0
    one_by_one, together = (B.fastgl_block_aggregate_fwd(ip, ix, wd, num_src, "gcn", x) for x in (aligned, moved))
    assert_close(host_feat(one_by_one, dtype), oracle.aggregate_fwd(blk.indptr, blk.indices, w, num_src, "gcn", dtype, X), dtype)
    assert torch.equal(one_by_one, together)


@pytest.mark.parametrize("dtype,feat", [("f32", 256), ("bf16", 512)])
@pytest.mark.parametrize("hot", [False, True])
def test_column_tiles_of_more_columns_than_have_their_scale_factors_in_l2(hot, dtype, feat):
    """One tile after the other where often read columns have a quarter of the edges, which only a plan with the transpose
    knows, else the tiles of a row together: the same bits, and a sample of rows against sums in fp64."""
    num_src, num_dst = (1 << 18) + 1, 40000
    rng = np.random.default_rng(feat + hot)
    lengths = rng.integers(0, 68, num_dst)
    lengths[:3] = 0, 256, 1000
    blk = block_of(lengths, num_src, 3)
    if hot:
        blk.indices[::2] = 2500 * rng.integers(0, 100, blk.indices[::2].size)
    assert column_tiles(blk, feat, dtype) == 2
    g = torch.Generator(device="cuda")
    g.manual_seed(feat)
    X = torch.randn((num_src, feat), generator=g, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    moved = torch.empty(X.numel() + 8, dtype=X.dtype, device="cuda")[8:].reshape(X.shape).copy_(X)
    ip, ix = dev_i32(blk.indptr), dev_i32(blk.indices)
    plan = B.fastgl_block_plan_create(ip, ix, num_src)
    assert (4 * B.lib().fastgl_long_row_chunk() * int(read_i32(plan, plan.export().counters, 4)[3]) >= blk.num_edges) == hot
    known = B.fastgl_block_aggregate_fwd(ip, ix, None, num_src, "gcn", X, plan=plan)
    for other in (B.fastgl_block_aggregate_fwd(ip, ix, None, num_src, "gcn", X),
                  B.fastgl_block_aggregate_fwd(ip, ix, None, num_src, "gcn", moved, plan=plan)):
        assert torch.equal(known, other)
    dout = np.bincount(blk.indices, minlength=num_src)
    for r in [0, 1, 2, 3, 63, 64, 20000, num_dst - 1]:
        cols = blk.indices[blk.indptr[r]:blk.indptr[r + 1]]
        scale = 1 / np.sqrt(max(1, cols.size) * dout[cols].astype(np.float64))
        terms = X[torch.from_numpy(cols.astype(np.int64)).cuda()].double() * torch.from_numpy(scale).cuda()[:, None]
        want, size = terms.sum(0), terms.abs().sum(0)
        # f32: weights rounded to fp32, fp64 sums, rounded once; bf16: fp32 products and sums, rounded to 8 bits
        bound = size * (cols.size + 4) * 2.0 ** -24 + want.abs() * (2.0 ** -23 if dtype == "f32" else 2.0 ** -8)
        assert ((known[r].double() - want).abs() <= bound).all(), r


@pytest.mark.parametrize("dtype,feat,weighted", [("f32", 100, False), ("f32", 125, True), ("bf16", 200, False)])
def test_many_wavefronts_of_two_groups(dtype, feat, weighted):
    """Enough rows for the variant with more gathers in flight (f32) and wavefronts of several row sets: rows of none to a
    few edges and every remainder of a batch."""
    blk = block_of(np.random.default_rng(feat).integers(0, 7, 300000), 5000, feat)
    check_block(blk, "mean", dtype, feat, weighted, True, feat, "many wavefronts")
