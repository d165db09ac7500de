"""Row walks at the widths where their kind changes (32 and 33 slices: lane groups or whole wavefronts; 64 and 65: one or
two column tiles), with no, one and two weights per edge, long rows whose chunks fill one or several ranges of the
reduction; and the one-kernel layer around the numbers of rows where a wavefront takes two or four of them (3 072, 6 144,
12 288, 18 432, 65 536).  Against the oracle, with the tolerances of the parity tests and of the layer's tests."""
import os
import re

import numpy as np
import pytest

import blockgen as bg
from test_gpu_layer import check_layer
from test_gpu_parity import check_block

pytestmark = pytest.mark.gpu
SOURCE = open(os.path.join(os.path.dirname(__file__), "..", "paper_2409_14939_amd", "csrc", "aggregate.hip")).read()


@pytest.mark.parametrize("mode,weighted", [("sum", False), ("mean", True), ("gcn", False), ("gcn", True)])
@pytest.mark.parametrize("feat,dtype", [(8, "f32"), (128, "f32"), (129, "f32"), (132, "f32"), (260, "f32"), (66, "f32"),
                                        (256, "bf16"), (264, "bf16"), (130, "bf16"), (33, "bf16"), (520, "bf16")])
def test_widths(feat, dtype, mode, weighted):
    rng = np.random.default_rng(feat)
    for hub in (129, 257, 128 * 9 + 1, 128 * 70):
        blk = bg.random_block(rng, 301, 517, 5.0, empty_frac=0.2, hub_rows=2, hub_deg=hub)
        check_block(blk, mode, dtype, feat, weighted, True, feat + hub, f"hub {hub}")


@pytest.mark.parametrize("feat,dtype,parts", [(256, "f32", 4), (128, "f32", 8), (602, "f32", 4), (40, "f32", 16), (5, "bf16", 64)])
def test_rows_of_few_and_of_many_chunks(feat, dtype, parts):
    """Long rows of one chunk less than a workgroup has groups to one more, some with a short last chunk, side by side, in
    both directions (every source that is used is used as often).  So few that each has a workgroup."""
    lengths = [257, 384, 385] + [128 * c + d for c in (parts - 1, parts, parts + 1, 2 * parts, 3 * parts + 1) for d in (-127, -1, 0) if 128 * c + d > 0]
    rng = np.random.default_rng(feat)
    deg = rng.permutation(np.concatenate([lengths, rng.integers(0, 4, 50)]))
    ip = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    src = rng.permutation(deg.size)[:deg.size // 2]
    ix = np.concatenate([np.repeat(src, deg[src]), rng.integers(0, deg.size, ip[-1])])[:ip[-1]]
    blk = bg.Block(ip, rng.permutation(ix).astype(np.int32), deg.size, deg.size)
    check_block(blk, "mean", dtype, feat, True, True, feat, "chunks")


def test_more_long_rows_than_one_pass_takes():
    """More (row, column tile) pairs than the groups of all workgroups together."""
    rng = np.random.default_rng(3)
    deg = np.where(np.arange(2900) % 700 == 5, 257 + 128 * 5, 257)
    ip = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    blk = bg.Block(ip, rng.integers(0, 3000, ip[-1]).astype(np.int32), deg.size, 3000)
    check_block(blk, "sum", "f32", 602, False, False, 3, "many long rows")


@pytest.mark.parametrize("feat,dtype,parts,tiles", [(256, "f32", 4, 1), (128, "f32", 8, 1), (602, "f32", 4, 3), (40, "f32", 16, 1),
                                                    (5, "bf16", 64, 1)])
def test_more_units_than_workgroups(feat, dtype, parts, tiles):
    """More than twice as many (row, column tile) units as workgroups, in both directions (a source is used as often as the row of its
    number has edges): rows of up to as many chunks as a workgroup has groups are added up by one group, several groups to a
    wavefront where rows are narrow; of those with more a workgroup has several on its list."""
    blocks = int(re.search(r"kReduceBlocks = (\d+);", SOURCE).group(1))
    rows, apart = 2 * blocks // tiles + 60, blocks // tiles
    deg = np.full(rows, 257)
    at = 10
    for c in (parts - 1, parts, parts + 1, 2 * parts, 3 * parts + 1):
        for d in (-127, -1, 0):
            # the same workgroup's units: `blocks` of them apart
            deg[[at, at + apart - 1, at + apart, at + apart + 1]] = max(257, 128 * c + d)
            at += 3
    lists = np.repeat((deg + 127) // 128, tiles)[: 2 * blocks].reshape(2, blocks) > parts
    assert deg.min() > 256 and rows * tiles > 2 * blocks and (lists.sum(axis=0) == 2).sum() >= 9
    rng = np.random.default_rng(feat)
    ip = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    ix = rng.permutation(np.repeat(np.arange(rows), deg)).astype(np.int32)
    check_block(bg.Block(ip, ix, rows, rows), "mean", dtype, feat, True, True, feat, "units")


@pytest.mark.parametrize("rows", [1, 3, 4, 5, 2047, 2048, 2049, 2065, 3072, 3073, 3079, 6144, 6145, 6161, 12288, 12289, 18432, 18433, 65536, 65537])
@pytest.mark.parametrize("mode,K,N,weighted", [("gcn", 256, 47, False), ("gcn", 60, 64, True), ("sum", 4, 1, False)])
def test_layer_rows(rows, mode, K, N, weighted):
    rng = np.random.default_rng(rows + K)
    blk = bg.random_block(rng, rows, 2 * rows + 40, 9.0, empty_frac=0.1)
    check_layer(blk, mode, K, N, True, weighted, True, True, rows + K, "rows")
