"""The static tile schedule of the join kernel, enumerated on the host (csrc/tile_cursor.h compiled with g++):
every tile of the triangle (self-join) or grid (two sets) exactly once, workgroups of an XCD balanced to within
one tile and, step by step, on at most two of the XCD's 8 x 4 rectangles."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build_schedule(tmp_path_factory, kind):
    out = tmp_path_factory.mktemp("sched") / f"libsched_{kind}.so"
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2508_21230_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "schedule_dump.cpp"), "-o", str(out)]
    if kind == "rowmajor_ablation":
        cmd.insert(1, "-DEJOIN_ABL_ROWMAJOR_TILES")
    if kind == "no_fast_path":
        cmd.insert(1, "-DEJOIN_CURSOR_NO_FAST_PATH")
    subprocess.run(cmd, check=True)
    lib = ctypes.CDLL(str(out))
    lib.ejoin_test_schedule.restype = ctypes.c_int64
    lib.ejoin_test_schedule.argtypes = [ctypes.c_uint32] * 4 + [ctypes.c_void_p, ctypes.c_int64]
    lib.ejoin_test_schedule_rows.restype = ctypes.c_int64
    lib.ejoin_test_schedule_rows.argtypes = [ctypes.c_uint32] * 6 + [ctypes.c_void_p, ctypes.c_int64]

    def run(nblocks, self_join, nt_a, nt_b):
        want = nt_a * (nt_a + 1) // 2 if self_join else nt_a * nt_b
        buf = np.zeros((want + 8, 4), dtype=np.uint32)
        m = lib.ejoin_test_schedule(nblocks, int(self_join), nt_a, nt_b, buf.ctypes.data, want + 8)
        return buf[:min(m, want + 8)], m, want
    def run_rows(nblocks, self_join, nt_a, nt_b, row_begin, row_end):
        want = nt_a * (nt_a + 1) // 2 if self_join else nt_a * nt_b
        buf = np.zeros((want + 8, 4), dtype=np.uint32)
        m = lib.ejoin_test_schedule_rows(nblocks, int(self_join), nt_a, nt_b, row_begin, row_end, buf.ctypes.data, want + 8)
        return buf[:min(m, want + 8)], m
    lib.ejoin_test_strips.restype = ctypes.c_int64
    lib.ejoin_test_strips.argtypes = [ctypes.c_uint32] * 5 + [ctypes.c_void_p, ctypes.c_int64]

    def run_strips(nblocks, self_join, stages, panels_begin, panels_end):
        buf = np.zeros((400 * nblocks, 4), dtype=np.uint32)
        m = lib.ejoin_test_strips(nblocks, int(self_join), stages, panels_begin, panels_end, buf.ctypes.data, len(buf))
        assert m <= len(buf)
        return buf[:m].astype(np.int64)
    lib.ejoin_test_strip_plan.restype = ctypes.c_int32
    lib.ejoin_test_strip_plan.argtypes = [ctypes.c_int32, ctypes.c_int64, ctypes.c_int64] + [ctypes.c_int32] * 3
    lib.ejoin_test_once.argtypes = [ctypes.c_uint32] * 4 + [ctypes.c_void_p]
    run.once = lib.ejoin_test_once
    run.kind = kind
    run.plan = lib.ejoin_test_strip_plan
    run.rows = run_rows
    run.strips = run_strips
    return run


@pytest.fixture(scope="module", params=["xcd_rectangles", "rowmajor_ablation"])
def sched(request, tmp_path_factory):
    return build_schedule(tmp_path_factory, request.param)


CASES = [(256, True, t, t) for t in (1, 2, 3, 15, 16, 17, 31, 32, 33, 40, 100, 391)] + \
        [(256, False, a, b) for a, b in ((1, 1), (1, 50), (50, 1), (7, 9), (16, 16), (17, 33), (391, 4), (4, 391), (100, 77))] + \
        [(8, True, 20, 20), (64, True, 45, 45), (304, True, 60, 60), (24, False, 30, 11), (250, True, 130, 130)]


@pytest.mark.parametrize("nblocks,self_join,nt_a,nt_b", CASES)
def test_every_tile_exactly_once(sched, nblocks, self_join, nt_a, nt_b):
    tiles, m, want = sched(nblocks, self_join, nt_a, nt_b)
    assert m == want
    I, J = tiles[:, 2].astype(np.int64), tiles[:, 3].astype(np.int64)
    assert (I < nt_a).all() and (J < nt_b).all()
    if self_join:
        assert (I <= J).all()
    keys = I * (nt_b + 1) + J
    assert np.unique(keys).size == want


@pytest.mark.parametrize("nblocks,self_join,nt_a,nt_b", [c for c in CASES if c[0] == 256])
def test_workgroups_of_an_xcd_stay_together(sched, nblocks, self_join, nt_a, nt_b):
    if sched.kind != "xcd_rectangles":
        pytest.skip("property of the XCD-aware schedule only")
    tiles, m, want = sched(nblocks, self_join, nt_a, nt_b)
    blk, step, I, J = (tiles[:, k].astype(np.int64) for k in range(4))
    xcd = blk % 8
    for x in range(8):
        sel = xcd == x
        counts = np.bincount(blk[sel] // 8, minlength=nblocks // 8)
        assert counts.max() - counts.min() <= 1, "tiles per workgroup of one XCD differ by more than one"
        for s in range(int(step[sel].max()) + 1 if sel.any() else 0):
            now = sel & (step == s)
            # the 8 x 4 rectangle a tile belongs to: (super-block, position inside it)
            rect = set(zip((I[now] // 8).tolist(), (J[now] // 4).tolist()))

            def full(r):  # all 32 cells of the rectangle are tiles of the problem
                i0, j0 = 8 * r[0], 4 * r[1]
                return i0 + 8 <= nt_a and j0 + 4 <= nt_b and (not self_join or i0 + 7 <= j0)
            # 32 consecutive entries of the XCD's list: one full rectangle, or the end of one and the start of the
            # next; partially empty rectangles (diagonal, ragged edge) hold fewer tiles, so more of them fit
            if all(full(r) for r in rect):
                assert len(rect) <= 2, f"XCD {x} step {s}: workgroups spread over {len(rect)} full rectangles"


@pytest.mark.parametrize("nblocks,self_join,nt_a,nt_b", CASES + [(256, True, 1000, 1000), (256, False, 700, 333), (256, True, 784, 784),
                                                                 (248, True, 500, 500), (256, False, 48, 1600)])
def test_fast_step_gives_the_same_sequence_as_the_general_step(tmp_path_factory, nblocks, self_join, nt_a, nt_b):
    """The cursor's shortcut for runs of complete rectangles is an optimisation only: workgroup by workgroup, step by
    step, it yields the tiles the general enumeration yields."""
    global _pair
    try:
        fast, slow = _pair
    except NameError:
        _pair = fast, slow = build_schedule(tmp_path_factory, "xcd_rectangles"), build_schedule(tmp_path_factory, "no_fast_path")
    a, ma, want = fast(nblocks, self_join, nt_a, nt_b)
    b, mb, _ = slow(nblocks, self_join, nt_a, nt_b)
    assert ma == mb == want
    assert np.array_equal(a, b)


@pytest.mark.parametrize("self_join,nt_a,nt_b,cuts", [(True, 100, 100, (0, 2, 3, 7)), (True, 391, 391, (0, 5, 11, 18, 25)), (False, 50, 77, (0, 1, 4)),
                                                     (True, 17, 17, (0, 1, 2)), (True, 40, 40, (0, 9))])
def test_launches_cut_by_rows_of_super_blocks_cover_every_tile_once(sched, self_join, nt_a, nt_b, cuts):
    """A join returned in batches runs one launch per range of super-block rows: the ranges' tiles are disjoint and
    together are all the tiles."""
    if sched.kind != "xcd_rectangles":
        pytest.skip("the row-major ablation enumerates the whole grid in one launch")
    want = nt_a * (nt_a + 1) // 2 if self_join else nt_a * nt_b
    bounds = list(cuts) + [0xFFFFFFFF]
    keys = []
    for lo, hi in zip(bounds[:-1], bounds[1:]):
        tiles, m = sched.rows(256, self_join, nt_a, nt_b, lo, hi)
        I, J = tiles[:, 2].astype(np.int64), tiles[:, 3].astype(np.int64)
        assert m == len(tiles)
        assert ((I // 16 >= lo) & (I // 16 < hi)).all()
        keys.append(I * (nt_b + 1) + J)
    keys = np.concatenate(keys)
    assert keys.size == want and np.unique(keys).size == want


@pytest.mark.parametrize("nblocks,self_join,nt_a,nt_b", [c for c in CASES if c[0] == 256] + [(256, True, 79, 79), (256, False, 118, 28), (256, False, 782, 2)])
def test_every_workgroup_gets_the_same_number_of_tiles(sched, nblocks, self_join, nt_a, nt_b):
    """Over the whole chip, not only inside an XCD; and a workgroup that goes on inside a band stays in its row."""
    if sched.kind != "xcd_rectangles":
        pytest.skip("property of the XCD-aware schedule only")
    tiles, m, want = sched(nblocks, self_join, nt_a, nt_b)
    counts = np.bincount(tiles[:, 0], minlength=nblocks)
    assert counts.max() == -(-want // nblocks) and counts.min() == want // nblocks
    blk, I, J = (tiles[:, k].astype(np.int64) for k in (0, 2, 3))
    off_diagonal = J >= (I // 8 + 1) * 8 if self_join else np.ones(m, dtype=bool)
    on = (blk[1:] == blk[:-1]) & (I[1:] // 8 == I[:-1] // 8) & off_diagonal[1:] & off_diagonal[:-1] & ((I[1:] // 8 + 1) * 8 <= nt_a)
    assert (I[1:][on] == I[:-1][on]).all() and (J[1:][on] == J[:-1][on] + nblocks // 8).all()


@pytest.mark.parametrize("nblocks,self_join,n_a,n_b", [(256, True, n, n) for n in (1, 64, 65, 512, 513, 5000, 20011, 100000)] +
                         [(256, False, a, b) for a, b in ((1, 1), (500, 200000), (200000, 500), (7001, 30011), (513, 64), (70000, 900))] +
                         [(7, True, 9000, 9000), (24, False, 30000, 5000), (300, True, 40000, 40000), (64, False, 100, 100000)])
def test_strips_cover_every_stage_once_and_evenly(sched, nblocks, self_join, n_a, n_b):
    """Runs of 64-column stages in panels of 512 rows: every stage right of the diagonal once, cut into launches or not, and (grids of
    whole XCDs) no workgroup with more than a few stages over its share."""
    panels, stages = (n_a + 511) // 512, (n_b + 63) // 64
    for cuts in ([0, panels], [0, min(8, panels), panels] if self_join else [0, panels]):
        seen = np.zeros((panels, stages), dtype=np.int64)
        load = np.zeros(nblocks, dtype=np.int64)
        for begin, end in zip(cuts[:-1], cuts[1:]):
            runs = sched.strips(nblocks, self_join, stages, begin, end)
            assert ((runs[:, 1] >= begin) & (runs[:, 1] < end) & (runs[:, 2] < runs[:, 3]) & (runs[:, 3] <= stages)).all()
            for b, panel, c, c_end in runs:
                seen[panel, c:c_end] += 1
                load[b] += c_end - c
        want = np.arange(stages)[None, :] >= 8 * np.arange(panels)[:, None] if self_join else np.ones_like(seen, dtype=bool)
        assert np.array_equal(seen, want.astype(np.int64))
        if nblocks == 256 and len(cuts) == 2:
            assert load.max() <= -(-load.sum() // 256) + 2


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return build_schedule(tmp_path_factory, "xcd_rectangles").plan


@pytest.mark.parametrize("nkb", range(2, 8))
def test_larger_self_joins_of_few_coordinates_have_no_gap(plan, nkb):
    """Lists and counts alike, from 27,000 points on."""
    rng = np.random.default_rng(nkb)
    for n in np.concatenate([np.arange(27000, 140000, 511), np.exp(rng.uniform(np.log(140000), np.log(5e8), 300)).astype(np.int64)]):
        assert plan(256, int(n), int(n), 1, nkb, 0) == plan(256, int(n), int(n), 1, nkb, 1) == 1, n


def test_counts_of_two_large_sets_of_few_coordinates_have_no_gap_either(plan):
    for n in range(20000, 200000, 3001):
        for nkb in range(2, 8):
            assert all(plan(256, a, b, 0, nkb, count) for a, b in ((n, 500000), (500000, n)) for count in (0, 1)), (n, nkb)


@pytest.mark.parametrize("nkb", range(2, 11))
def test_two_sets_are_joined_alike_whichever_comes_first(plan, nkb):
    """Lists: the same kernel, and the same set in its rows.  Counts: the points, each with more hits the more queries there are, in the
    rows where the queries are many times as many."""
    rng = np.random.default_rng(nkb)
    for a, b in np.exp(rng.uniform(np.log(300), np.log(600000), (4000, 2))).astype(np.int64).tolist() + [(700, 100000), (300, 300000)]:
        if (a + 63) // 64 == (b + 63) // 64:
            continue
        assert (plan(256, a, b, 0, nkb, 0), plan(256, b, a, 0, nkb, 0)) in ((0, 0), (1, 3), (3, 1)), (a, b)
        assert 16 * min(a, b) > max(a, b) or plan(256, min(a, b), max(a, b), 0, nkb, 1) in (0, 1), (a, b)


@pytest.mark.parametrize("nkb", [8, 9])
def test_self_counts_with_the_filter_in_the_open_go_there_from_large_sets_on(plan, nkb):
    rule = [plan(256, n, n, 1, nkb, 1) for n in range(20000, 400000, 997)]
    assert not any(rule[:80]) and all(rule[160:])  # up to 99,000 points, from 179,000 on
    assert all(plan(256, n, n, 1, nkb, 0) for n in range(60000, 400000, 997))  # lists


@pytest.mark.parametrize("self_join,nt_a,nt_b", [(True, n, n) for n in (1, 2, 5, 38)] + [(False, a, b) for a, b in ((1, 1), (1, 9), (9, 1), (2, 2), (7, 30), (30, 7))])
def test_the_one_launch_join_has_every_tile_once_and_those_that_others_wait_for_first(sched, self_join, nt_a, nt_b):
    tiles = nt_a * (nt_a + 1) // 2 if self_join else nt_a * nt_b
    out = np.zeros((tiles, 2), dtype=np.uint32)
    sched.once(tiles, int(self_join), nt_a, nt_b, out.ctypes.data)
    want = {(i, j) for i in range(nt_a) for j in range(i if self_join else 0, nt_b)}
    assert {tuple(t) for t in out.tolist()} == want
    first = nt_a if self_join else nt_a + nt_b - 1
    assert all(i == j if self_join else i == 0 or j == 0 for i, j in out[:first].tolist())
