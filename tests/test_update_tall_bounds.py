"""Host-side model of what the tall tiles of the update phase (csrc/update_rows.hip, k_update_tall) move through
buffers: an access whose offset is at or past the buffer's size is dropped (a store) or gives 0 (a load).
Results: a tile's rows past the last one are not masked, only dropped that way; no element outside the result may
survive, for any remainder of rows and columns and either element size.  Column operand (W of the forward pass): rows
past the last one are not masked either; every one of their elements must come back as 0.  Rows loaded eight elements
at a time (load_at, load_oct, buffer_oct; the small tiles have no buffer around them): every load lies inside its row,
or, for rows of odd length in bf16, in the aligned dword that holds the row's last element.  Look-ahead: which chunks of A
and stages of B the loop asks for, and that it multiplies the right ones.  The model mirrors the kernel's index arithmetic
and takes its constants from the source; it has to be changed with it."""
import os
import random
import re

import numpy as np

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2409_14939_amd", "csrc")
SOURCE = "".join(open(os.path.join(CSRC, name)).read() for name in ("update_rows.hip", "update_tall_turn.inc"))


def constant(name):
    text = re.search(rf"constexpr \w+ {name} = ([^;]+);", SOURCE).group(1)
    return eval(re.sub(r"\(int64_t\)|u\b", "", re.sub(r"(0x[0-9A-Fa-f]+)u", r"\1", text)))


TALL_ROWS, FULL = constant("kTallRows"), constant("kFull")
NOWHERE, MAX_LD, STAGE_ELEMS = constant("kNowhere"), constant("kMaxTallLd"), constant("kStageElems")
# the lines of the kernel that `fetches` repeats
LOOP = ("KS = NT < 64 ? 64 : kStageElems / NT", "AHEAD = !BF16 && (NTILES == 4 || (GATE && NTILES == 8)) ? 1 : 2;",
        "TURN = AHEAD == 1 && KS <= 32 ? 32 : 64;", "load_b(0);", "load_a(i, 32 * i);", "stage_b(0, 0);", "int lk = KS;",
        "for (; k0 + TURN < Kc; k0 += TURN) turn(std::false_type(), k0);",
        "turn(std::true_type(), k0);", "for (int k0 = 0; k0 < Kc; k0 += TURN) {", "for (int step = 0; step < TURN / 16; ++step) {",
        "kc = k0 + 32 * cc, from = cc % AHEAD;", "if (LAST && step > 0 && k0 + 16 * step >= Kc) break;", "if (16 * step % KS == 0) {",
        "stage_b(cur ^ 1, lk);", "lk += KS;", "if (s == 0) load_a(from, kc + 32 * AHEAD);", "slot = 16 * step % KS / 8 + h;",
        "if (16 * (step + 1) % KS == 0) {", "row = arow + (k0 < Kc ? 0u : kNowhere);",
        "buffer_cols<VB>(rb, (uint32_t)(k0 + 8 * bs) * ldb + bcol, ldb, bcols);")
LIMIT = "(b_col && (g.Kc + 64) * g.ldb >= (int64_t)1 << 29)"


def fetches(nt, bf16, gate, Kc):
    """(first indices of the chunks of A, first indices of the stages of B, indices of a stage) that the loop asks for; asserts
    that a step of 16 is multiplied out of the chunk and the stage that hold it."""
    ks = 64 if 32 * nt < 64 else STAGE_ELEMS // (32 * nt)
    ahead = 1 if not bf16 and (nt == 4 or (gate and nt == 8)) else 2
    turn = 32 if ahead == 1 and ks <= 32 else 64
    a, b = [32 * i for i in range(ahead)], [0, ks]
    chunk, lds, loaded, cur, multiplied = list(a), [0, None], ks, 0, []
    for k0 in range(0, Kc, turn):
        for step in range(turn // 16):
            kc = k0 + 32 * (step >> 1)
            src = (step >> 1) % ahead
            if step > 0 and k0 + 16 * step >= Kc:
                break
            if step & 1 == 0:
                taken = chunk[src]
            if 16 * step % ks == 0:
                lds[cur ^ 1] = loaded
                loaded += ks
                b.append(loaded)
            if step & 1 == 0:
                chunk[src] = kc + 32 * ahead
                a.append(chunk[src])
            assert taken == kc and lds[cur] + 16 * step % ks == k0 + 16 * step
            multiplied.append(k0 + 16 * step)
            if 16 * (step + 1) % ks == 0:
                cur ^= 1
    assert multiplied == list(range(0, Kc, 16))
    return a, b, ks


FORMS = [(nt, bf16, gate) for nt in (1, 2, 4, 8) for bf16 in (False, True) for gate in (False, True)]


def rows_ahead(Kc):
    """Rows of a column operand past its last one that the loop asks for, at most."""
    return max(max(b) + ks for b, ks in (fetches(*f, Kc)[1:] for f in FORMS)) - Kc


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
    """Elements of the rows K, K + 1, ... that the loop asks for: all at or past the buffer's end."""
    row, col = np.meshgrid(np.arange(K, K + rows_ahead(K)), np.arange(256), indexing="ij")
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


def test_the_kernel_has_the_loop_that_the_model_repeats():
    for line in LOOP + (LIMIT,):
        assert line in SOURCE, line


def test_the_loop_multiplies_every_step_out_of_what_it_loaded():
    for form in FORMS:
        for Kc in list(range(1, 200)) + [256, 601, 602, 1024]:
            fetches(*form, Kc)


def test_look_ahead_past_the_last_index_wraps_around_nowhere():
    """Chunks of A past the end start at kNowhere, stages of B past the end behind the last row: both have to stay between
    every buffer's end (at most 2^31 - 1 bytes) and 2^32, for the longest rows and the largest column operands that the
    tall tiles take."""
    size = (1 << 31) - 1
    for eb in (2, 4):
        last = (TALL_ROWS - 1) * MAX_LD * eb + MAX_LD * eb + 15          # the row's last element, the load that holds it
        assert NOWHERE > size and NOWHERE + last < 1 << 32
    most = max(rows_ahead(Kc) for Kc in range(1, 300))
    assert 64 < most <= 192                                              # the model sees more than one stage ahead
    for ldb in (1, 3, 256, 257, MAX_LD):
        Kc = ((1 << 29) - 1) // ldb - 64                                 # the most that LIMIT lets through
        if Kc < 1:
            continue
        assert (Kc + 64) * ldb < 1 << 29 <= (Kc + 65) * ldb
        assert Kc * ldb * 4 <= size and (Kc + most) * ldb * 4 + 8 < 1 << 32
