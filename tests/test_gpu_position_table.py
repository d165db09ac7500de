"""Tables whose slots hold input positions (hash_table.h) at the sizes where their rules change: one, two and many
positions (bits left for the hash), more blocks of 1024 IDs than a ranking workgroup adds up itself (4096), and
around the number of mini-batches whose overlaps are counted from marks (4, 8).  Whole numbers: equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2409_14939_amd import binding as B

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int64)).cuda()


@pytest.mark.parametrize("n_dst,n_nbr", [(1, 1), (1, 2), (2, 3), (1023, 1), (1024, 1025), (700_000, 4096 * 1024 - 700_000),
                                         (700_001, 4096 * 1024 - 700_000)])
def test_idmap_sizes(n_dst, n_nbr):
    print(f"case idmap n_dst={n_dst} n_nbr={n_nbr}", flush=True)
    rng = np.random.default_rng(n_dst + n_nbr)
    ids = rng.permutation(2 * n_dst + 8).astype(np.int64) * 0x5DEECE66D + 11
    dst, nbr = ids[:n_dst], ids[(rng.random(n_nbr) ** 2 * ids.size).astype(np.int64)]
    ref_local, ref_uniq = oracle.idmap(dst, nbr)
    local, uniq, res = B.fastgl_idmap(dev(dst), dev(nbr), "ordered")
    assert res.tolist() == [ref_uniq.size, 0]
    assert np.array_equal(local.cpu().numpy(), ref_local)
    assert np.array_equal(uniq.cpu().numpy()[:ref_uniq.size], ref_uniq)
    local, uniq, res = B.fastgl_idmap(dev(dst), dev(nbr), "fused")
    local, uniq = local.cpu().numpy(), uniq.cpu().numpy()[:ref_uniq.size]
    assert res.tolist() == [ref_uniq.size, 0] and np.array_equal(uniq[:n_dst], dst)
    assert np.array_equal(np.sort(uniq), np.sort(ref_uniq)) and np.array_equal(uniq[local], nbr)


@pytest.mark.parametrize("n_prev,n_new", [(1, 1), (2, 1024), (1025, 3), (5000, 4096 * 1024), (5000, 4096 * 1024 + 1)])
def test_match_sizes(n_prev, n_new):
    print(f"case match n_prev={n_prev} n_new={n_new}", flush=True)
    rng = np.random.default_rng(n_prev + n_new)
    ids = rng.permutation(n_prev + n_new).astype(np.int64) * 0x5DEECE66D + 11
    prev, new = ids[:n_prev], rng.permutation(ids)[:n_new]
    src_row, load_pos, load_gid, res = B.fastgl_match(dev(prev), dev(new))
    row_of = {int(g): r for r, g in enumerate(prev)}
    want = np.fromiter((row_of.get(int(g), -1) for g in new), np.int64, n_new)
    miss = np.flatnonzero(want < 0)
    want[miss] = -1 - np.arange(miss.size)
    assert res.tolist() == [miss.size, 0]
    assert np.array_equal(src_row.cpu().numpy(), want)
    assert np.array_equal(load_pos.cpu().numpy()[:miss.size], miss)
    assert np.array_equal(load_gid.cpu().numpy()[:miss.size], new[miss])


@pytest.mark.parametrize("n", [1, 2, 4, 5, 8, 9, 64])
def test_overlap_counts(n):
    print(f"case overlap of {n} mini-batches", flush=True)
    rng = np.random.default_rng(n)
    pool = rng.permutation(6000).astype(np.int64) * 0x5DEECE66D + 11
    sets = [rng.permutation(pool)[:int(rng.integers(0, 3000))] for _ in range(n)]
    offsets = np.concatenate([[0], np.cumsum([s.size for s in sets])])
    gid = np.concatenate(sets)
    counts, viol = B.fastgl_overlap_counts(dev(gid), offsets.tolist())
    assert int(viol) == 0 and np.array_equal(counts.cpu().numpy().reshape(n, n), oracle.overlap_matrix(sets))
    bad = gid.copy()                                    # one repeated and one negative ID
    bad[offsets[n] - 1], bad[offsets[n] - 2] = bad[offsets[n] - 3], -5
    if sets[-1].size >= 3:
        assert int(B.fastgl_overlap_counts(dev(bad), offsets.tolist())[1]) == 2
