"""Host-side model of what the tall tiles of the update phase (csrc/update_rows.hip, k_update_tall) move through
buffers: an access whose offset is at or past the buffer's size is dropped (a store) or gives 0 (a load).
Results: a tile's rows past the last one are not masked, only dropped that way; no element outside the result may
survive, for any remainder of rows and columns and either element size.  Column operand (W of the forward pass): rows
past the last one are not masked either; every one of their elements must come back as 0.  Rows loaded eight elements
at a time (load_at, load_oct, buffer_oct; the small tiles have no buffer around them): every load lies inside its row,
or, for rows of odd length in bf16, in the aligned dword that holds the row's last element.  The model mirrors the kernel's index arithmetic; it has to be changed with it."""
import random

import numpy as np

TALL_ROWS, FULL = 128, 240


def tall_tiles(M, N, b_col):
    rows = -(-M // TALL_ROWS)
    if b_col and N <= 32:
        return 1
    best, best_cost = 2, -(-N // 64) * 64 * 20
    for nt in (4, 8):
        tiles = -(-N // (32 * nt))
        cost = tiles * 32 * nt * (17 if nt == 4 else 16)
        if rows * tiles >= FULL and cost <= best_cost:
            best, best_cost = nt, cost
    return best


def exact(nbytes):
    return nbytes


def whole_dwords(nbytes):
    return (nbytes + 3) & ~3


def stores_in_bounds(M, N, eb, b_col, size=exact):
    nt = 32 * tall_tiles(M, N, b_col)
    r0 = (M - 1) // TALL_ROWS * TALL_ROWS                     # the last row tile: the others hold whole rows
    row, col = np.meshgrid(np.arange(TALL_ROWS), np.arange(nt), indexing="ij")
    for c0 in {0, (N - 1) // nt * nt}:
        off = (row * N + col) * eb
        kept = (c0 + col < N) & (off < size(((M - r0) * N - c0) * eb))
        if not np.array_equal(kept, (r0 + row < M) & (c0 + col < N)):
            return False
    return True


def column_operand_ends(K, N, eb, size=exact):
    """Elements of the rows K, K + 1, ... that a stage of 64 contracted indices and the one ahead of it may ask for."""
    row, col = np.meshgrid(np.arange(K, K + 128), np.arange(256), indexing="ij")
    return not ((row * N + col) * eb < size(K * N * eb)).any()


def shapes():
    rng = random.Random(5)
    yield from [(17001, 61), (9003, 101), (31001, 255), (17000, 47), (16385, 1), (31000, 256)]
    for _ in range(200):
        yield rng.randint(16385, 40000), rng.randint(1, 300)


def test_tall_tiles_store_their_result_and_nothing_else():
    for M, N in shapes():
        for eb in (2, 4):
            for b_col in (False, True):
                assert stores_in_bounds(M, N, eb, b_col), (M, N, eb, b_col)


def test_the_model_sees_a_size_rounded_up():
    """The mistake the model exists for: a size rounded up to a dword lets the bf16 element behind the result through."""
    assert not stores_in_bounds(17001, 61, 2, True, whole_dwords)
    assert not stores_in_bounds(9003, 101, 2, False, whole_dwords)


def test_rows_of_a_column_operand_past_the_last_one_are_zero():
    for K, N in [(101, 47), (33, 9), (17, 255), (100, 256), (1, 1)]:
        for eb in (2, 4):
            assert column_operand_ends(K, N, eb), (K, N, eb)
    assert not column_operand_ends(101, 47, 2, whole_dwords)


def row_load_bytes(V, k, K, row):
    """[first, last] byte of the loads of elements k .. k + 7 of a row of K elements that starts at byte `row`."""
    if V == 4:                                                # fp32: two quads
        at = [min(k + 4 * i, K - 4) for i in range(2)]
        return row + 4 * min(at), row + 4 * max(at) + 15
    if V == 8:                                                # bf16, rows of whole dwords
        at = row + 2 * min(k, K - 8)
        return at, at + 15
    if V == 9:                                                # bf16, odd rows: the five dwords around eight elements
        at = row + 2 * min(k, K - 8)
        base = at & ~3
        return base, base + (16 if at & 2 else 12) + 3
    eb = 4 if V == 1 else 2                                   # element by element
    at = [k + i if k + i < K else 0 for i in range(8)]
    return row + eb * min(at), row + eb * max(at) + eb - 1


def test_row_loads_stay_inside_their_rows():
    for V, eb, lengths in ((4, 4, range(4, 70)), (8, 2, range(8, 70, 2)), (9, 2, range(9, 70, 2)), (1, 4, range(1, 20)), (2, 2, range(1, 70))):
        for K in lengths:
            for r in range(3):                                # the third row is the matrix's last
                row, end = r * K * eb, 3 * K * eb
                for k in range(0, K + 128, 8):
                    first, last = row_load_bytes(V, k, K, row)
                    if V == 9:
                        assert first >= 0 and last < whole_dwords(row + K * eb) <= whole_dwords(end), (V, K, r, k)
                    else:
                        assert row <= first and last < row + K * eb, (V, K, r, k)


def test_offsets_inside_a_tile_fit_32_bits():
    """Rows of up to 2^21 elements: the last element that a tile of 256 rows may ask for lies below 2^31 bytes."""
    assert 255 * (1 << 21) * 4 + (1 << 21) * 4 - 1 < 1 << 31


def test_look_ahead_past_the_last_index_wraps_around_nowhere():
    """Chunks of A past the end start 2^31 bytes further on; a stage of B and the two after it ask for up to 190 rows past
    the last one.  Both have to stay between every buffer's end (at most 2^31 - 1 bytes) and 2^32."""
    far = 127 * (1 << 21) * 4 + (1 << 21) * 4 + 15
    assert (1 << 31) + far < 1 << 32
    for ldb in (1, 3, 256, 1 << 21):
        Kc = ((1 << 29) - 1) // ldb - 64                      # the longest that the tall tiles take
        assert (Kc + 64) * ldb < 1 << 29 and (Kc + 191) * ldb * 4 + ldb * 4 < 1 << 32
