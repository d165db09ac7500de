"""GPU parity of the overlap counts of windows of many IDs, which go through buckets: the sizes where the path, the number of
buckets and the size of a bucket's table change, one to eight mini-batches, buckets that overflow their tables, IDs that are
negative or repeated.  Whole numbers: everything is compared exactly."""
import numpy as np
import pytest
import torch

import oracle
from paper_2409_14939_amd import binding as B

pytestmark = pytest.mark.gpu
LINE, LINE_MANY = 7 << 16, 3 << 16   # IDs from which the buckets are used: up to four mini-batches, more
ODD = np.uint64(0x9E3779B97F4A7C15)     # of near_hash


def counted(sets):
    offsets = np.concatenate([[0], np.cumsum([len(s) for s in sets])])
    print(f"case overlaps of {len(sets)} mini-batches, {offsets[-1]} IDs", flush=True)
    gid = torch.from_numpy(np.concatenate(sets)).cuda()
    counts, violations = B.fastgl_overlap_counts(gid, offsets.tolist())
    return counts.cpu().numpy(), int(violations.cpu()[0])


def window(rng, sizes, span):
    """Mini-batches of the given sizes, each about half of it from a common pool."""
    pool = np.unique(rng.integers(0, span, size=max(sizes) + 1))
    sets = []
    for m in sizes:
        own = np.unique(np.concatenate([pool[rng.random(pool.size) < 0.5], rng.integers(0, span, size=m)]))
        sets.append(rng.permutation(own)[:m])
    return sets


def expected(sets):
    """The oracle's answer; of large windows in one pass over their distinct IDs, which is quicker."""
    if sum(map(len, sets)) < 4 << 20:
        return oracle.overlap_matrix(sets)
    distinct, at = np.unique(np.concatenate(sets), return_inverse=True)
    holds = np.zeros((len(sets), distinct.size), np.float32)
    for row, part in zip(holds, np.split(at, np.cumsum([len(s) for s in sets])[:-1])):
        row[part] = 1.0
    return np.array([[np.count_nonzero(a * b) for b in holds] for a in holds])


def ids_of(hashes):
    """The IDs with these hashes (uint64): near_hash backwards."""
    x = hashes * np.uint64(pow(int(ODD), -1, 2 ** 64))
    far = (x >> np.uint64(22)) * ODD
    return (x ^ (far ^ far >> np.uint64(32)) * ODD >> np.uint64(42)).astype(np.int64)


def crowd(rng, count, bits):
    """Distinct IDs whose hashes agree in the upper `bits` bits, in random order."""
    h = rng.integers(0, 2 ** (64 - bits), size=3 * count).astype(np.uint64) | np.uint64(0xA5 << (64 - bits))
    ids = np.unique(ids_of(h))
    return rng.permutation(ids[ids >= 0])[:count]


@pytest.mark.parametrize("total,n", [(LINE - 1, 4), (LINE, 4), (LINE + 1, 1), (LINE_MANY - 1, 5), (LINE_MANY, 8), (LINE_MANY, 5),
                                     (2400 * 256, 2), (2400 * 256 + 1, 8), (2400 * 512 + 1, 5), (2400 * 1024 + 1, 3), (2560 * 2048, 4),
                                     (2560 * 2048 + 1, 8), (2560 * 2048 + 1, 3), (12 << 20, 4), ((12 << 20) + 1, 4)])
def test_sizes(total, n):
    rng = np.random.default_rng(total + n)
    cuts = np.sort(rng.integers(total // (2 * n), total, size=n - 1)) if n > 1 else np.array([], np.int64)
    sets = window(rng, np.diff(np.concatenate([[0], cuts, [total]])).tolist(), 4 * total if n % 2 else 2 ** 45)
    fill = total - sum(len(s) for s in sets)               # IDs that no pool has
    sets[-1] = np.concatenate([sets[-1], 2 ** 50 + np.arange(fill)])
    counts, violations = counted(sets)
    assert violations == 0 and np.array_equal(counts, expected(sets))


@pytest.mark.parametrize("in_one", [3000, 3072, 3073, 3100, 30_000])
def test_a_bucket_that_overflows(in_one):
    """Distinct IDs whose hashes agree in the upper 8 bits, all in one bucket: within a table's room, just beyond, far beyond."""
    rng = np.random.default_rng(in_one)
    same = crowd(rng, in_one, 8)
    others = rng.permutation(np.unique(rng.integers(0, 2 ** 40, size=LINE)))
    sets = [np.concatenate([same, others[:100_000]]), np.concatenate([others[50_000:250_000], same[: in_one // 2]])]
    sets[1] = np.concatenate([sets[1], 2 ** 50 + np.arange(max(0, LINE - sum(map(len, sets))))])
    counts, violations = counted(sets)
    assert violations == 0 and np.array_equal(counts, expected(sets))


@pytest.mark.parametrize("in_one,bits,total,n", [(10_000, 8, LINE_MANY, 8), (7000, 11, 2560 * 2048 + 1, 3), (20_000, 11, 2560 * 2048 + 1, 8)])
def test_overflow_with_more_mini_batches_and_large_tables(in_one, bits, total, n):
    """Every mini-batch holds its own half of the crowded IDs; a table holds 3 072 of them, a large one 7 168."""
    rng = np.random.default_rng(in_one + n)
    same = crowd(rng, in_one, bits)
    pool = rng.permutation(total)[: 2 * total // n] + 2 ** 50
    sets = [np.concatenate([rng.permutation(same)[: in_one // 2], rng.permutation(pool)[: total // n - in_one // 2 + 1]]) for _ in range(n)]
    assert sum(map(len, sets)) >= total
    counts, violations = counted(sets)
    assert violations == 0 and np.array_equal(counts, expected(sets))


@pytest.mark.parametrize("count", [16_385, LINE // 4])
@pytest.mark.parametrize("stride", [832_040, 14_930_352, 267_914_296, 2 ** 20, 2 ** 40 + 1])
def test_multiples_of_a_number(stride, count):
    rng = np.random.default_rng(7)
    sets = [rng.permutation(2 * count)[:count].astype(np.int64) * stride for _ in range(4)]
    counts, violations = counted(sets)
    assert violations == 0 and np.array_equal(counts, expected(sets))


def test_negative_and_repeated_ids_are_counted():
    rng = np.random.default_rng(5)
    a, b = window(rng, [LINE, LINE], 2 ** 40)
    a, b = a[:200_000], b[:200_000]
    expect = oracle.overlap_matrix([a, b])
    counts, violations = counted([np.concatenate([a, a[:777], [-1, -(2 ** 63)]]), np.concatenate([b, [-5]])])
    assert violations == 780 and np.array_equal(counts, expect)
    counts, violations = counted([np.full(LINE, 12345), np.array([12345, 6])])      # one bucket has them all
    assert violations == LINE - 1 and counts.tolist() == [[1, 1], [1, 2]]
    counts, violations = counted([np.full(LINE, -1)])
    assert violations == LINE and counts.tolist() == [[0]]
