"""Host-side model of every global load address of the tiled update kernel (csrc/update.hip: PlaneMover
and HalfMover init / fetch and run_steps), checked against the extents of the operands: no
lane of any workgroup may read outside [0, numel) of the matrix it loads from, including the masked
lanes (which load from the step's first row) and the look-ahead fetch of the step
after the last one.  The row products' own kernels: test_update_tall_bounds.py.  The model mirrors the kernel's
index arithmetic line by line; it has to be changed with it."""
import random

import numpy as np

K_TILE, K_STEP = 128, 16


def clamp4(n):
    return np.clip(n, 0, 4)


def slab_rows(M, K, N):
    tiles = (max((K + 127) // 128, 1) if K > 0 else 1) * ((N + 127) // 128)
    best, best_cost = 32, None
    for rows in range(32, 2049, 32):
        nslab = (max(M, 1) + rows - 1) // rows
        rounds = (nslab * tiles + 767) // 768
        cost = rounds * (rows * 156250 + 20000000) + nslab * (K * N + N) * 2
        if best_cost is None or cost < best_cost:
            best, best_cost = rows, cost
    return best


def fetches_of(kbeg, kend, quads):
    """(first contracted index, masked) of every fetch of run_steps."""
    length = max(kend - kbeg, 0)
    nstep = (length + K_STEP - 1) // K_STEP if length > 0 else 1
    plain = max(0, length // K_STEP - 1) if quads else 0
    assert plain < nstep
    return [(kbeg, True)] + [(kbeg + K_STEP * (i + 1), i >= plain) for i in range(nstep)]


def operand_in_bounds(quads, numel, ld, o0, omax, kbeg, kend, origin_of_missing_step=0):
    t = np.arange(256)
    o = o0 + 4 * (t & 31)
    at = np.minimum(o, omax - 4) if quads else o
    for k, mask in fetches_of(kbeg, kend, quads):
        origin = (k if k < kend else origin_of_missing_step) * ld
        for s in range(2):
            off = (2 * (t >> 5) + s) * ld + at
            ok = (k + 2 * (t >> 5) + s < kend) if mask else np.full(256, True)
            if quads:                     # four elements at off, or in the step's first row
                lo = origin + np.where(ok, off, at)
                hi = lo + 3
                # columns that exist come from their own place: column o + j is element j + moved of the quad
                moved = np.minimum(o - at, 3)
                for j in range(4):
                    exists = o + j < omax
                    assert (moved[exists] + j <= 3).all() and (at[exists] + moved[exists] == o[exists]).all()
            else:                         # element i < n at off + i, the others at the step's first element
                n = np.where(ok, clamp4(omax - o), 0)
                lo = np.minimum(origin + np.where(n > 0, off, 0), origin)
                hi = np.maximum(origin + np.where(n > 0, off + n - 1, 0), origin)
            if lo.min() < 0 or hi.max() >= numel:
                return False
    return True


def weight_gradient_in_bounds(M, K, N, **kw):
    """dW: H [M][K] and dZ [M][N], contracted over slabs of M."""
    slab, quads = slab_rows(M, K, N), K >= 4 and N >= 4
    ranges = [(b, min(b + slab, M)) for b in range(0, M, slab)]
    ok = True
    for kb, ke in (ranges[0], ranges[-1]):
        for r0 in {0, (K - 1) // K_TILE * K_TILE}:
            ok &= operand_in_bounds(quads, M * K, K, r0, K, kb, ke, **kw)
        for c0 in {0, (N - 1) // K_TILE * K_TILE}:
            ok &= operand_in_bounds(quads, M * N, N, c0, N, kb, ke, **kw)
    return ok


SHAPES = [(512345, 100, 256), (91331, 256, 256), (8000, 256, 47), (91331, 1024, 256), (1, 1, 1), (5, 3, 2),
          (129, 17, 130), (300, 100, 47), (1000, 33, 64), (128, 16, 128), (128, 32, 128), (256, 48, 256), (77, 80, 4),
          (4096, 64, 128)]


def test_every_load_of_the_update_kernel_stays_inside_its_operand():
    rng = random.Random(1)
    shapes = SHAPES + [(rng.randint(1, 700), rng.randint(1, 300), rng.randint(1, 300)) for _ in range(200)]
    for M, K, N in shapes:
        assert weight_gradient_in_bounds(M, K, N), (M, K, N)


def half_tile_in_bounds(M, N, quads, slab, first_row_of_missing_step=0):
    """dY as the operand of 64 columns (N <= 64): two columns of two contracted rows per lane."""
    t = np.arange(256)
    o = 2 * (t & 31)
    at = np.minimum(o, N - 2) if quads else o
    for kbeg, kend in {(0, min(slab, M)), ((M - 1) // slab * slab, M)}:
        for k, mask in fetches_of(kbeg, kend, quads):
            origin = (k if k < kend else first_row_of_missing_step) * N
            for s in range(2):
                off = (2 * (t >> 5) + s) * N + at
                ok = (k + 2 * (t >> 5) + s < kend) if mask else np.full(256, True)
                if quads:
                    first = origin + np.where(ok, off, at)
                    last = first + 1
                else:
                    n = np.where(ok, np.clip(N - o, 0, 2), 0)
                    first = np.full(256, origin)
                    last = origin + np.maximum(np.where(n > 0, off, 0), np.where(n > 1, off + 1, 0))
                if first.min() < 0 or last.max() >= M * N:
                    return False
    return True


def test_every_load_of_the_narrow_tile_stays_inside_its_operand():
    rng = random.Random(2)
    shapes = [(1150398, 64), (8000, 47), (1, 9), (31, 10), (33, 32), (1001, 64), (16, 64), (17, 12)]
    for M, N in shapes + [(rng.randint(1, 700), rng.randint(9, 64)) for _ in range(200)]:
        for quads in (True, False):
            assert half_tile_in_bounds(M, N, quads, slab_rows(M, 100, N)), (M, N, quads)
    assert not half_tile_in_bounds(1001, 64, True, slab_rows(1001, 100, 64), 1001)


def test_the_model_sees_a_fetch_past_the_last_step():
    """The mistake the model exists for: taking the origin of a step beyond the range from that
    step's own index reads past the end of the operand."""
    M, K, N = 100, 100, 256
    assert not operand_in_bounds(True, M * N, N, 0, N, 0, M, origin_of_missing_step=112)
