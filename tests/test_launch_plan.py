"""The host's launch decisions for a call (no GPU), from per-segment counts
only: teams per workgroup, the tile kernel's grid, the number of workers that
the work queue is cut for, its capacity, and whether the sums of several
entries of a segment meet (finalize).  Where they do, the tile partials and the
row counts are zeroed first, and an open call ends with the zeroing pass; a
one-tile segment whose tile were cut without that would get a wrong tag, so it
must be so whenever the expansion kernel's cut can reach a one-tile segment.
And how many workgroups share a record of a token call."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2608_25431_amd import gift

THREADS, ROWS = 1024, 128
PIECE_ROWS = ROWS // 4


class QueuePlan(ctypes.Structure):
    _fields_ = [("cap", ctypes.c_uint64), ("grid", ctypes.c_uint32), ("finalize", ctypes.c_bool)]


class TilePlan(ctypes.Structure):
    _fields_ = [("teams", ctypes.c_uint32), ("grid", ctypes.c_uint32), ("workers", ctypes.c_uint32), ("q", QueuePlan)]


def symbol(prefix):
    """An internal function of the library, by its mangled name's prefix."""
    if not os.path.exists(gift.LIB_PATH):
        from paper_2608_25431_amd import build
        build.build()
    lib = gift.lib()
    out = subprocess.run(["nm", "-D", "--defined-only", gift.LIB_PATH], capture_output=True, text=True).stdout
    names = [l.split()[-1] for l in out.splitlines() if l.strip()]
    return getattr(lib, next(n for n in names if n.startswith(prefix)))


def plan_tiles_function():
    """plan_tiles(n_tiles, rows of all tiles, segments of several tiles, most rows of a one-tile segment, CUs, open)."""
    fn = symbol("_ZN4gift10plan_tiles")
    fn.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_bool]
    fn.restype = TilePlan
    return fn


@pytest.fixture(scope="module")
def plan_queue():
    fn = symbol("_ZN4gift10plan_queue")
    fn.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint32]
    fn.restype = QueuePlan
    return fn


def can_cut_one_tile(n_tiles, rows_all, one_rows_max, cus):
    """Whether the expansion kernel's rule can cut the tile of a one-tile
    segment with one_rows_max rows: with fewer tiles than CUs it cuts tiles
    of more than ceil(rows_all / cus) rows (none when that is a whole tile or
    more); otherwise only tiles of more than PIECE_ROWS rows."""
    if n_tiles < cus:
        p = -(-rows_all // cus)
        return p < ROWS and one_rows_max > p
    return one_rows_max > PIECE_ROWS


@pytest.mark.parametrize("cus", [256, 64, 7, 1])
def test_plan_covers_the_kernel_rule(plan_queue, cus):
    r = np.random.default_rng(cus)
    for _ in range(400):
        n_one = int(r.integers(0, 40))
        n_multi = int(r.integers(0, 3)) if r.random() < 0.5 else 0
        one_rows = r.integers(1, ROWS + 1, n_one)
        multi_tiles = r.integers(2, 12, n_multi)
        multi_first = r.integers(1, ROWS + 1, n_multi)
        n_tiles = n_one + int(multi_tiles.sum())
        rows_all = int(one_rows.sum()) + int(((multi_tiles - 1) * ROWS + multi_first).sum())
        one_max = int(one_rows.max()) if n_one else 0
        q = plan_queue(n_tiles, rows_all, n_multi, one_max, cus)
        if n_tiles == 0:
            assert (q.cap, q.grid, q.finalize) == (0, 0, False)
            continue
        assert q.cap == n_tiles + (ROWS // PIECE_ROWS - 1) * cus
        assert 1 <= q.grid <= cus
        # enough workgroups for every entry up to one per CU
        assert q.grid >= min(cus, n_tiles)
        need = n_multi > 0 or can_cut_one_tile(n_tiles, rows_all, one_max, cus)
        assert q.finalize == need


def a_call(r, cus):
    """Tile count, rows, multi-tile segments and the most rows of a one-tile segment of a random table, its tile count
    around one and two per CU and its rows around the plan's lines often."""
    n = int(r.choice([0, 1, 2, cus // 2, cus - 1, cus, cus + 1, 2 * cus - 1, 2 * cus, 2 * cus + 1, 3 * cus, 5 * cus]))
    n = max(0, n + int(r.integers(-1, 2)))
    mean = int(r.choice([1, 2, 7, 8, 15, 16, 17, 31, 32, 33, 64, ROWS]))
    one = np.full(n, mean) if r.random() < 0.5 else r.integers(1, mean + 1, n)
    if n and r.random() < 0.5:
        p = -(-int(one.sum()) // int(r.choice([1, cus, 2 * cus])))
        one[int(r.integers(0, n))] = np.clip(p + int(r.integers(-1, 5)), 1, ROWS)
    tiles = r.integers(2, 5, int(r.integers(1, 3))) if r.random() < 0.3 else np.zeros(0, int)
    rows = int(one.sum()) + int(((tiles - 1) * ROWS).sum()) + int(r.integers(1, ROWS + 1, len(tiles)).sum())
    return n + int(tiles.sum()), rows, len(tiles), int(one.max(initial=0))


@pytest.mark.parametrize("opened", [False, True])
@pytest.mark.parametrize("cus", [256, 64, 7, 1])
def test_tile_plan_covers_the_kernel_rule(cus, opened):
    plan_tiles, r = plan_tiles_function(), np.random.default_rng(cus)
    met = set()
    for _ in range(3000):
        n_tiles, rows, n_multi, one_max = a_call(r, cus)
        t = plan_tiles(n_tiles, rows, n_multi, one_max, cus, opened)
        if n_tiles == 0:
            assert (t.q.cap, t.q.finalize) == (0, False)
            continue
        # how the kernel runs it
        two = rows <= (7 if 2 * cus < n_tiles <= 3 * cus else 16) * n_tiles if n_tiles > cus else rows <= cus
        assert t.teams == (2 if two else 1)
        w = t.teams * cus if n_tiles > cus else cus
        assert t.workers in (1, w + (n_tiles == w))  # cut evenly also with a tile for each
        assert min(cus, n_tiles) <= t.grid <= cus
        # the queue for that many workers: its capacity, and whether the cut can give a segment several entries
        assert t.q.cap == n_tiles + (ROWS // PIECE_ROWS - 1) * t.workers
        assert t.q.finalize == (n_multi > 0 or can_cut_one_tile(n_tiles, rows, one_max, t.workers))
        # one worker stands for an uncut queue, where a cut would not pay
        if t.workers == 1 and cus > 1:
            assert not t.q.finalize and one_max <= PIECE_ROWS
            assert n_tiles >= w or one_max < -(-rows // w) + (3 if opened else 2)
        met.add((t.teams, t.workers, t.q.finalize))
    assert cus == 1 or met >= {(1, 1, False), (2, 1, False), (1, cus, True), (2, cus, True), (2, 2 * cus, True)}


def test_examples(plan_queue):
    # one 1.5 MiB segment on 256 CUs: cut into one-row pieces, tag from the last of them
    q = plan_queue(1, 96, 0, 96, 256)
    assert q.finalize and q.grid == 96
    # 256 short one-tile segments: nothing to cut, no sums meet
    q = plan_queue(256, 256 * 4, 0, 4, 256)
    assert not q.finalize and q.grid == 256
    # more one-tile segments than CUs, longer than a quarter tile: the tail cut can reach them
    q = plan_queue(300, 300 * 96, 0, 96, 256)
    assert q.finalize and q.grid == 256


@pytest.fixture(scope="module")
def token_shift():
    fn = symbol("_ZN4gift11token_shift")
    fn.argtypes = [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint64]
    fn.restype = ctypes.c_uint32
    return lambda segs, chunks: fn(segs.ctypes.data, len(segs), chunks)


@pytest.mark.parametrize("counts", [[64 * 4096], [1] * 5000, [64 * 64] * 64, [64 * 9 - 3] * 300, [1 << 24],
                                    [1 << 16] + [1] * 1024, [100] * 3000, [1 << 30, 1]])
def test_token_records(token_shift, counts):
    """Token records shared by 1 << shift workgroups of 64 tokens: at most an eighth of the workgroups find no tokens,
    and twice as many could not share without that (or the table is small).  The work of a workgroup stays 64 tokens,
    however long the call."""
    segs = np.zeros(len(counts), gift.SEGMENT_DTYPE)
    segs["row_count"] = counts
    chunks = [-(-c // 64) for c in counts]

    def records(shift):
        return sum(-(-c // (1 << shift)) for c in chunks)
    n = sum(chunks)
    s = token_shift(segs, n)
    assert records(s) << s <= n + n // 8
    assert records(s) <= 16 or s == 16 or records(s + 1) << (s + 1) > n + n // 8


def test_few_chunks_are_not_shared(token_shift):
    segs = np.zeros(1, gift.SEGMENT_DTYPE)
    segs["row_count"] = 64 * 2048
    assert token_shift(segs, 2048) == 0
