"""Plans of small blocks, which are built in one launch: bit for bit against the oracle at the edges of what that
launch takes (and just beyond, where the staged build takes over), and small blocks built in stages together
with a large one."""
import numpy as np
import pytest
import torch

import blockgen as bg
import oracle
from paper_2409_14939_amd import binding as B
from gpu_util import dev_i32, read_f32, read_i32
from test_gpu_parity import check_bookkeeping

pytestmark = pytest.mark.gpu


def exact_block(rng, num_dst, num_src, edges, hub=0):
    """`edges` edges over the rows at random, `hub` of them in one row; sources skewed to low ids."""
    cuts = np.sort(rng.integers(0, edges - hub + 1, num_dst - 1)) if num_dst > 1 else np.zeros(0, np.int64)
    deg = np.diff(np.concatenate([[0], cuts, [edges - hub]]))
    deg[rng.integers(num_dst)] += hub
    idx = np.minimum((rng.random(edges) ** 2 * num_src).astype(np.int64), num_src - 1)
    blk = bg.Block(np.concatenate([[0], np.cumsum(deg)]).astype(np.int32), idx.astype(np.int32), num_dst, num_src)
    blk.check()
    return blk


@pytest.mark.parametrize("nd,ns,edges,hub", [(1, 1, 1, 0), (3, 2048, 64, 0), (256, 2049, 1025, 300), (24576, 40000, 65535, 0),
                                             (24577, 40000, 65535, 0), (1000, 4097, 65536, 0), (70, 900, 65535, 60000),
                                             (5000, 262144, 30000, 2000), (5000, 262145, 30000, 2000), (2000, 6000, 24577, 257)])
def test_plan_of_a_small_block(nd, ns, edges, hub):
    check_bookkeeping(exact_block(np.random.default_rng(nd + edges), nd, ns, edges, hub), "once")


def test_small_blocks_next_to_a_large_one_and_alone():
    rng = np.random.default_rng(5)
    small = [exact_block(rng, 100, 3000, 2500, 400), exact_block(rng, 4000, 9000, 9000)]
    # more workgroups of 512 sources than the device has compute units: 2 048 to a workgroup
    many = [exact_block(rng, 2000, 32768 - 2047 * i, 16000 + 97 * i, 300) for i in range(6)] + small
    many[3].indices[:13000] = rng.integers(4096, 6144, 13000)
    for blocks in (small, small + [exact_block(rng, 30000, 50000, 90000, 700)], many):
        dev = [(dev_i32(b.indptr), dev_i32(b.indices), b.num_src) for b in blocks]
        for blk, plan in zip(blocks, B.fastgl_block_plan_create_many(dev, B.PLAN_ALL | B.PLAN_PERM)):
            v = plan.export()
            pT, iT, perm = oracle.transpose(blk.indptr, blk.indices, blk.num_src)
            assert np.array_equal(read_i32(plan, v.indptr_T, blk.num_src + 1), pT)
            assert np.array_equal(read_i32(plan, v.indices_T, blk.num_edges), iT)
            assert np.array_equal(read_i32(plan, v.perm, blk.num_edges), perm)


@pytest.mark.parametrize("nd,ns,edges,hub", [(70, 900, 65535, 60000), (65536, 70000, 65535, 300), (65537, 70000, 3000, 0)])
def test_forward_only_plan_with_source_degrees(nd, ns, edges, hub):
    blk = exact_block(np.random.default_rng(nd), nd, ns, edges, hub)
    ip, ix = dev_i32(blk.indptr), dev_i32(blk.indices)
    plan = B.fastgl_block_plan_create(ip, ix, ns, B.PLAN_FWD | B.PLAN_SRC_DEG)
    v = plan.export()
    din, dout = oracle.degrees(blk.indptr, blk.indices, ns)
    assert np.array_equal(read_i32(plan, v.din, nd), din) and np.array_equal(read_i32(plan, v.dout, ns), dout)
    np.testing.assert_allclose(read_f32(plan, v.src_rsqrt, ns), 1.0 / np.sqrt(np.maximum(dout, 1)), rtol=1e-6)
    rows, cptr = oracle.long_rows(blk.indptr, B.fastgl_long_row_threshold(), B.fastgl_long_row_chunk())
    cnt = read_i32(plan, v.counters, 2)
    assert cnt[0] == rows.shape[0] and cnt[1] == cptr[-1]
    assert np.array_equal(read_i32(plan, v.long_dst, rows.shape[0]), rows)
    sp = oracle.work_split(blk.indptr, B.fastgl_work_per_group())
    assert np.array_equal(read_i32(plan, v.split_dst, sp.shape[0]), sp)
    torch.cuda.synchronize()


@pytest.mark.parametrize("edges", [16384, 16385, 20480, 20481])
def test_full_plan_around_the_edge_limit(edges):
    check_bookkeeping(exact_block(np.random.default_rng(edges), 3000, 4097, edges, 9000), "once")


# the limit of sparse blocks (at most four edges per source), buckets of 512 sources, several chunks of one bucket
@pytest.mark.parametrize("nd,ns,edges", [(300, 5119, 20480), (300, 5119, 20481), (300, 5120, 20480), (300, 5121, 20484), (9000, 12288, 49152),
                                         (9000, 12289, 49152), (9000, 12289, 49153), (9000, 12287, 49152), (700, 511, 20000),
                                         (700, 512, 20000), (700, 513, 20000), (700, 1024, 8192), (700, 1025, 8193)])
def test_full_plan_around_the_limit_of_sparse_blocks(nd, ns, edges):
    check_bookkeeping(exact_block(np.random.default_rng(ns + edges), nd, ns, edges, 500), "once")


# nearly all edges in one bucket of 512 sources (over all of them, over 64, over one): its chunks go to different
# workgroups; the other bucket gets just over a chunk where there is room.  Edges in the bucket: multiples of every power
# of two up to 32 768, and one more
@pytest.mark.parametrize("ns,bucket", [(12288, 0), (12288, 23), (32768, 63), (12800, 7)])
@pytest.mark.parametrize("inside", [8192, 8193, 16385, 32768, 40961, 49152])
def test_full_plan_of_a_block_with_one_full_bucket(ns, bucket, inside):
    rng = np.random.default_rng(ns + bucket + inside)
    blk = exact_block(rng, 5000, ns, 49152, 700)
    for i, spread in enumerate((512, 64, 1)):
        idx = 512 * ((bucket + 1) % (ns // 512)) + rng.integers(0, 512, 49152)
        idx[rng.permutation(49152)[:inside]] = 512 * bucket + 3 * i + rng.integers(0, spread, inside) % (512 - 3 * i)
        blk.indices[:] = idx
        blk.check()
        check_bookkeeping(blk, f"spread {spread}")


@pytest.mark.parametrize("nd,ns,edges,hub", [(3000, 32768, 16384, 300), (3000, 32769, 16384, 300), (24576, 32768, 16384, 300),
                                             (24577, 32768, 16384, 300), (100, 32768, 16384, 0)])
def test_full_plan_around_the_limits_of_rows_and_sources(nd, ns, edges, hub):
    blk = exact_block(np.random.default_rng(nd + ns), nd, ns, edges, hub)
    blk.indices[-900:] = ns - 1                                # the last source is a long row of the transpose
    check_bookkeeping(blk, "once")


@pytest.mark.parametrize("nd", [8192, 8193, 24576, 24577])
@pytest.mark.parametrize("parts", [B.PLAN_FWD, B.PLAN_FWD | B.PLAN_SRC_DEG])
def test_forward_only_plan_around_the_row_limits(nd, parts):
    ns, edges = 30000, 50000
    blk = exact_block(np.random.default_rng(nd), nd, ns, edges, 5000)
    plan = B.fastgl_block_plan_create(dev_i32(blk.indptr), dev_i32(blk.indices), ns, parts)
    v = plan.export()
    din, dout = oracle.degrees(blk.indptr, blk.indices, ns)
    assert np.array_equal(read_i32(plan, v.din, nd), din)
    if parts & B.PLAN_SRC_DEG:
        assert np.array_equal(read_i32(plan, v.dout, ns), dout)
    rows, cptr = oracle.long_rows(blk.indptr, B.fastgl_long_row_threshold(), B.fastgl_long_row_chunk())
    cnt = read_i32(plan, v.counters, 2)
    assert cnt[0] == rows.shape[0] and cnt[1] == cptr[-1]
    assert np.array_equal(read_i32(plan, v.long_dst, rows.shape[0]), rows)
