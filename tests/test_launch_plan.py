"""The launch planner (csrc/drot_plan.h) without a GPU: which kernel runs which sweep.

The product library enqueues exactly what this logic decides.  Here it is compiled with the host
compiler (libdrot_plan.so) and driven with scripted statuses: every path, every switch between paths
(zero-segment skipping <-> even/odd pairs, 8-wave screened <-> lean), continued calls, the early looks
at the density, a stop at a check with work queued behind it.
"""
import ctypes
import os

import numpy as np
import pytest

RESIDENT, PRO32, PLAIN32, TALL64, SCREENED8, LEAN, POINTS, SLAB, TWOPASS, POINTS_LEAN = range(10)
NO_UPDATE, SEPARATE, MERGED_SLAB, MERGED_TILES = range(4)
COLS = ("sweep", "mode", "first", "prev_sums", "lines_in", "refresh", "pro", "tilesum", "update", "ra", "kind", "flags")
FRESH_CARRY = (0, -1000000, -1, 8, 0, 0, 0, 0)  # (what is left out of a carry is 0)


@pytest.fixture(scope="module")
def planlib():
    from paper_2305_18483_amd import build

    csrc = os.path.dirname(build.PLAN_SOURCE)
    sources = (build.PLAN_SOURCE, os.path.join(csrc, "drot_plan.h"), os.path.join(csrc, "drot_bounds.h"))
    if not os.path.exists(build.PLAN_LIB_PATH) or os.path.getmtime(build.PLAN_LIB_PATH) < max(map(os.path.getmtime, sources)):
        build.build_plan()
    lib = ctypes.CDLL(build.PLAN_LIB_PATH)
    lib.drot_plan_trace.restype = ctypes.c_int
    lib.drot_plan_labels.restype = ctypes.c_int
    return lib


class Trace:
    def __init__(self, rows, statics, carry, iters):
        self.rows, self.statics, self.carry, self.iters = rows, statics, carry, iters

    def col(self, name):
        return [int(r[COLS.index(name)]) for r in self.rows]


def trace(lib, m, n, max_iters, reg_kind=0, from_points=0, warm=0, resume=0, weights=0, c_on_lines=1, x_on_lines=1,
          slab_k=0, nruns=0, feedback=1, checking=1, check_every=100, resident=-1, fused_update=-1, skip_cost=-1,
          skip_unchanged=-1, screening=-1, nontemporal=-1, force_two_pass=0, gap_every=0, densities=(), lines=None,
          stop_at_status=-1, carry=FRESH_CARRY, line_bounds=None, rho=0):
    # (a handle holds the bounds by line, the fixed workspace, whose schedule has no feedback, does not)
    line_bounds = feedback if line_bounds is None else line_bounds
    problem = (ctypes.c_int * 16)(m, n, reg_kind, from_points, warm, resume, weights, c_on_lines, x_on_lines, slab_k, nruns,
                                  feedback, checking, max_iters, line_bounds, rho)
    options = (ctypes.c_int * 9)(check_every, resident, fused_update, skip_cost, skip_unchanged, screening, nontemporal,
                                 force_two_pass, gap_every)
    carry_io = (ctypes.c_longlong * 12)(*carry)
    dens = (ctypes.c_double * max(1, len(densities)))(*densities)
    assert lines is None or len(lines) == len(densities)
    nz_lines = None if lines is None else (ctypes.c_double * max(1, len(lines)))(*lines)
    cap = max_iters + 8
    rows = (ctypes.c_int * (12 * cap))()
    statics = (ctypes.c_int * 10)()
    iters = ctypes.c_int()
    nrows = lib.drot_plan_trace(problem, options, carry_io, dens, nz_lines, len(densities), stop_at_status, rows, cap,
                                statics, ctypes.byref(iters))
    assert nrows >= 0
    arr = np.array(rows[:12 * nrows], dtype=np.int64).reshape(nrows, 12)
    names = ("nseg", "ntr", "resident", "pad_c", "pad_x", "small", "fused", "may_screen", "adaptive", "nt")
    return Trace(arr, dict(zip(names, statics)), tuple(carry_io), iters.value)


def test_the_five_configurations_take_their_paths(planlib):
    t = trace(planlib, 100, 100, 2000, checking=0)
    assert t.statics["resident"] and t.col("sweep") == [RESIDENT] and len(t.rows) == 1  # one launch for all 2000
    t = trace(planlib, 100, 100, 250, checking=1, check_every=100)
    assert t.col("sweep") == [RESIDENT] * 3  # a launch per stretch between checks
    t = trace(planlib, 1000, 1000, 300, reg_kind=1)
    assert t.statics["small"] and t.statics["fused"] and not t.statics["adaptive"] and not t.statics["nt"]
    assert t.col("sweep")[0] == PLAIN32 and set(t.col("sweep")[1:]) <= {PRO32, PLAIN32}
    # one launch per iteration: the update runs separately only at the end of a stretch
    assert [i for i, u in enumerate(t.col("update")) if u == SEPARATE] == [99, 199, 299]
    assert t.col("sweep")[100] == PLAIN32 and t.col("sweep")[101] == PRO32  # after a materialised state: plain again
    t = trace(planlib, 20000, 20000, 40, reg_kind=1, checking=0)
    assert t.statics["may_screen"] and t.statics["adaptive"] and t.statics["nt"] and not t.statics["small"]
    t = trace(planlib, 5000, 5000, 30, reg_kind=2, slab_k=4, nruns=10)
    assert set(t.col("sweep")) == {SLAB} and set(t.col("update")) == {MERGED_SLAB} and not t.statics["small"]
    t = trace(planlib, 5000, 5000, 5, reg_kind=2, slab_k=0, nruns=5000)
    assert set(t.col("sweep")) == {TWOPASS} and set(t.col("update")) == {SEPARATE}


def test_padded_copies_when_rows_are_off_the_128_byte_lines(planlib):
    assert not trace(planlib, 300, 512, 1).statics["pad_c"] and not trace(planlib, 300, 512, 1).statics["pad_x"]
    s = trace(planlib, 300, 500, 1).statics
    assert s["pad_c"] and s["pad_x"]
    s = trace(planlib, 300, 512, 1, c_on_lines=0).statics
    assert s["pad_c"] and not s["pad_x"]
    s = trace(planlib, 300, 512, 1, x_on_lines=0).statics
    assert not s["pad_c"] and s["pad_x"]
    assert trace(planlib, 300, 512, 1, weights=1).statics["pad_c"]          # C + W needs a working copy
    s = trace(planlib, 300, 500, 1, from_points=1).statics
    assert not s["pad_c"] and s["pad_x"]                                     # no stored cost to pad
    s = trace(planlib, 100, 100, 1, x_on_lines=0, c_on_lines=0).statics
    assert s["resident"] and not s["pad_c"] and not s["pad_x"]               # the resident kernel takes any pitch


def test_cold_start_of_a_large_problem_moves_to_lines_after_two_epochs_of_bounds(planlib):
    t = trace(planlib, 20000, 20000, 300, reg_kind=1, checking=1, densities=(0.9, 0.6, 0.2, 0.05), lines=(0.3, 0.1, 0.04, 0.03))
    kinds = t.col("kind")
    # sweep 1 has nothing to read; sweeps 2 and 8 record the bounds, the sweep by lines runs from 9 on whatever the density,
    # on the line flags that sweep 8 leaves, and renews by itself
    assert kinds == [0, 6] + [5] * 5 + [6] + [7] * 292
    assert t.col("lines_in") == [0] * 8 + [1] * 292
    ends = [i + 1 for i, f in enumerate(t.col("flags")) if f & 1]
    assert ends[:6] == [16, 32, 64, 96, 100, 128]
    assert [bool(t.col("flags")[e - 1] & 2) for e in ends[:6]] == [True, True, True, True, False, True]
    assert set(t.col("update")[1:]) == {MERGED_TILES} and t.col("update")[0] == SEPARATE
    # column partials: 625 rows for the 32-row tiles, 313 in groups of four for the 64-row tiles, 79 for the lean sweep
    assert t.col("ra")[0] == 625 * 16 + 1 and t.col("ra")[5] == 313 * 16 + 4 and t.col("ra")[100] == 79 * 16 + 1
    assert set(t.col("mode")) == {0}
    assert t.carry[8] == 1 and t.carry[9] == 1 and t.carry[6] == 1  # by lines, drift and line flags as a continued call finds them
    # a third of the lines nonzero in nearly all row segments: still by lines; with a period that was asked for, sooner
    t = trace(planlib, 20000, 20000, 700, reg_kind=1, checking=1, densities=(0.95,), lines=(0.34,))
    assert set(t.col("kind")[8:]) == {7}
    t = trace(planlib, 20000, 20000, 30, reg_kind=1, checking=1, screening=3, densities=(0.95,), lines=(0.34,))
    assert t.col("kind")[:8] == [0, 6, 5, 5, 6, 7, 7, 7]


def test_dense_lines_go_to_the_even_odd_pairs_and_come_back(planlib):
    # statuses 0 .. 21 end the looks of the first 512 iterations and the checks among them, then there is one every 100
    steps = [(1.0, 0.97)] * 22 + [(0.99, 0.4)] * 3 + [(0.89, 0.4)]
    t = trace(planlib, 20000, 20000, 1500, reg_kind=1, checking=1, densities=[d for d, _ in steps], lines=[x for _, x in steps])
    kinds = t.col("kind")
    # early looks start nothing; the check at 100, read while 101 .. 128 are queued, does (more than 85 % of the lines)
    assert set(kinds[8:128]) == {7} and kinds[128:130] == [1, 2]
    # back at a check that finds no more than 90 % of the row segments nonzero (its status is read while the next stretch is
    # queued): bounds first, then the lines
    back = kinds.index(6, 128)
    ends = [i + 1 for i, f in enumerate(t.col("flags")) if f & 1]
    assert ends[21] == 512 and set(kinds[128:back]) == {1, 2} and back == ends[26]
    assert set(kinds[back + 1:]) == {7} and t.col("lines_in")[back + 1] == 1
    # at an early look below 99.5 % (half of the lines, were they independent)
    steps = [(1.0, 0.97)] * 9 + [(0.996, 0.4), (0.994, 0.4)]
    t = trace(planlib, 20000, 20000, 500, reg_kind=1, checking=1, densities=[d for d, _ in steps], lines=[x for _, x in steps])
    kinds, ends = t.col("kind"), [i + 1 for i, f in enumerate(t.col("flags")) if f & 1]
    assert t.col("flags")[ends[10] - 1] & 2 and kinds.index(6, 128) == ends[11] and set(kinds[128:ends[11]]) == {1, 2}
    # between 85 and 92 % of the lines: pairs as well; below, the lines stay although no row segment is empty
    t = trace(planlib, 20000, 20000, 400, reg_kind=1, checking=1, densities=(1.0,), lines=(0.9,))
    assert set(t.col("kind")[128:]) == {1, 2}
    t = trace(planlib, 20000, 20000, 400, reg_kind=1, checking=1, densities=(1.0,), lines=(0.8,))
    assert set(t.col("kind")[8:]) == {7}
    # without the pairs, above 92 %: row segments, until lines pay again
    t = trace(planlib, 20000, 20000, 400, reg_kind=1, checking=1, skip_cost=0, densities=(1.0,), lines=(0.97,))
    assert set(t.col("kind")[8:128]) == {7} and 7 not in t.col("kind")[128:] and 5 in t.col("kind")[128:]


def test_cold_start_of_a_small_screened_problem_moves_to_the_lean_sweep(planlib):
    # (screened because it was asked for; below 11.5 million entries the sweep by lines waits for a sparse plan)
    # statuses: the looks after 16, 32, 64 ... iterations report 90 %, 60 %, 20 %, 5 % nonzero row segments
    t = trace(planlib, 2300, 2500, 300, reg_kind=1, checking=1, screening=1, densities=(0.9, 0.6, 0.2, 0.05))
    kinds = t.col("kind")
    # sweep 1 has nothing to read; sweep 2 records the bounds, then after 8, 16, 32 sweeps again
    assert kinds[:12] == [0, 6] + [5] * 7 + [6, 5, 5]
    assert kinds[25] == 6 and kinds[57] == 6
    flags = t.col("flags")
    ends = [i + 1 for i, f in enumerate(flags) if f & 1]
    assert ends[:6] == [16, 32, 64, 96, 100, 128]
    assert [bool(flags[e - 1] & 2) for e in ends[:6]] == [True, True, True, True, False, True]
    # the third status (after 64: 20 %) is read while the stretch to 96 is queued: lean from sweep 97 on
    first_lean = kinds.index(7)
    assert first_lean == 96 and set(kinds[96:]) == {7}
    assert t.col("lines_in")[96] == 0 and set(t.col("lines_in")[97:]) == {1}  # flags are valid from one lean sweep to the next
    assert set(t.col("update")[1:]) == {MERGED_TILES} and t.col("update")[0] == SEPARATE
    # column partials: 72 rows for the 32-row tiles, 36 in groups of four for the 64-row tiles, 9 for the lean sweep
    assert t.col("ra")[0] == 72 * 16 + 1 and t.col("ra")[5] == 36 * 16 + 4 and t.col("ra")[100] == 9 * 16 + 1
    # never the even/odd pairs here: the dense readings came from early looks
    assert set(t.col("mode")) == {0}


def test_the_lean_sweep_stays_within_its_32_bit_offsets(planlib):
    # 64 rows of a tile, 4 bytes an entry, counted from the tile's first row: up to 2^24 - 1 columns, rounded up to whole lines
    for n, fits in ((16777184, True), (16777185, False), (17200000, False)):
        t = trace(planlib, 64, n, 130, reg_kind=1, checking=0, densities=(0.05,), lines=(0.01,))
        assert (7 in t.col("kind")) == fits and 6 in t.col("kind"), n


def test_gap_pass_goes_lean_once_bounds_and_flags_describe_the_plan(planlib):
    # stretch ends of the cold starts above: no bounds after the first sweeps of a call; row-segment sums serve as
    # flags after the 8-wave sweeps, the line flags after lean sweeps; never on paths that do not screen
    t = trace(planlib, 20000, 20000, 300, reg_kind=1, checking=1, check_every=100, densities=(0.9, 0.6, 0.2, 0.02))
    assert all(f & 8 and f & 16 for f in t.col("flags") if f & 1)
    t = trace(planlib, 2300, 2500, 300, reg_kind=1, checking=1, check_every=100, screening=1, densities=(0.9, 0.6, 0.2, 0.02))
    flags = t.col("flags")
    ends = {i + 1: f for i, f in enumerate(flags) if f & 1}
    assert all(f & 8 for f in ends.values())  # (bounds exist from sweep 2 on)
    assert not ends[16] & 16 and not ends[96] & 16 and ends[100] & 16 and ends[300] & 16
    t = trace(planlib, 1000, 1000, 200, reg_kind=1, checking=1, check_every=100)
    assert not any(f & 8 for f in t.col("flags"))
    t = trace(planlib, 20000, 20000, 200, reg_kind=1, checking=1, check_every=100, from_points=1)
    assert not any(f & 8 for f in t.col("flags"))
    t = trace(planlib, 5000, 5000, 200, reg_kind=2, slab_k=4, nruns=10, checking=1, check_every=100)
    assert not any(f & 8 for f in t.col("flags"))
    # even/odd pairs: the sums of a plain sweep at the stretch end still describe X, the bounds are those of the
    # last refresh
    t = trace(planlib, 20000, 20000, 64, reg_kind=1, checking=0, skip_unchanged=0)
    assert not any(f & 8 for f in t.col("flags"))  # (nothing recorded bounds)


def test_dense_plans_switch_to_the_even_odd_pairs_and_back(planlib):
    t = trace(planlib, 2300, 1500, 90, reg_kind=1, checking=0, check_every=10, screening=1, densities=(0.95,))
    kinds = t.col("kind")
    assert kinds[:10] == [0, 6] + [5] * 7 + [6]
    # early looks (16, 32, ...) never start the pairs; the status of the stretch ending at 10 does, read during 10..16
    assert set(kinds[16:]) == {1, 2} and kinds[10:16] == [5] * 6
    modes = t.col("mode")
    for end in [i + 1 for i, f in enumerate(t.col("flags")) if f & 1]:
        assert modes[end - 1] in (0, 2)  # X is plain at every stretch end
    # and back below 50 %
    t = trace(planlib, 2300, 1500, 80, reg_kind=1, checking=1, check_every=10, screening=0, resume=1,
              carry=(1, 900000, -1, 8, 1, 256, 0, 100), densities=(0.9, 0.4))
    kinds = t.col("kind")
    assert set(kinds[:30]) == {1, 2} and set(kinds[30:]) == {4}
    assert t.col("prev_sums")[30] == 1  # a mode-2 sweep leaves plain X and its sums


def test_odd_stretches_of_pairs_start_with_a_plain_sweep(planlib):
    t = trace(planlib, 700, 1300, 37, reg_kind=1, checking=1, check_every=7, fused_update=0, skip_cost=1)
    assert t.col("mode")[:7] == [0, 1, 2, 1, 2, 1, 2] and t.col("first")[0] == 1
    t = trace(planlib, 700, 1300, 8, reg_kind=1, checking=0, fused_update=0, skip_cost=1)
    assert t.col("mode") == [1, 2] * 4


def test_a_continued_call_goes_on_where_the_last_one_stopped(planlib):
    kw = dict(reg_kind=1, checking=1, check_every=50, densities=(0.9, 0.5, 0.1, 0.05, 0.05, 0.05))
    one = trace(planlib, 20000, 20000, 260, **kw)
    first = trace(planlib, 20000, 20000, 150, **kw)
    assert first.carry[4] == 1 and first.carry[6] == 1 and first.carry[7] == 150 and first.carry[2] >= 0
    second = trace(planlib, 20000, 20000, 110, resume=1, carry=first.carry, reg_kind=1, checking=1, check_every=50,
                   densities=(0.05,))
    # no new epoch, no dense first sweep: lean from its first sweep, line flags valid
    assert second.col("kind")[0] == 7 and second.col("lines_in")[0] == 1 and second.col("first")[0] == 0
    assert one.col("kind")[150:] == second.col("kind")
    # without continuation state (another option set, say) nothing is taken for granted
    cold = trace(planlib, 20000, 20000, 10, resume=1, carry=(0, 50000, -1, 8, 0, 0, 0, 150), reg_kind=1)
    assert cold.col("prev_sums")[0] == 0 and cold.col("kind")[0] == 6


def test_bounds_go_on_only_to_calls_with_the_cost_and_the_stepsize_they_were_recorded_with(planlib):
    # a solve over point clouds leaves bounds without the bounds by line, a stored-cost one none of the sweep's own costs;
    # both are of varphi - rho C: where the next call's cost comes from elsewhere, or its stepsize is another, it renews first
    handle = dict(reg_kind=1, checking=0)
    points = dict(handle, from_points=1, rho=50000, densities=(0.9, 0.6, 0.2, 0.05))
    stored = dict(handle, from_points=0, rho=50000, densities=(0.9, 0.6, 0.2, 0.05))
    lean_kind, full_kind = {0: 7, 1: 8}, {0: 6, 1: 9}
    for first, second in ((points, stored), (stored, points), (points, dict(points, rho=25000)),
                          (stored, dict(stored, rho=25000)), (points, points), (stored, stored)):
        a = trace(planlib, 20000, 20000, 500, **first)
        assert a.carry[2] > 0 and a.carry[4] == 1  # bounds, and sums that describe the plan
        b = trace(planlib, 20000, 20000, 60, resume=1, carry=a.carry, **dict(second, densities=(0.05,)))
        kinds = b.col("kind")
        lean = kinds.index(lean_kind[second["from_points"]])
        same = first["from_points"] == second["from_points"] and first["rho"] == second["rho"]
        assert (lean == 0) == same
        if not same:  # nothing certified before a sweep of this call has recorded the bounds
            assert full_kind[second["from_points"]] in kinds[:lean] and 5 not in kinds[:lean]


def test_what_the_certificates_of_the_sweep_by_lines_pass_stays_zero(planlib):
    # four columns of a line or row segment with x = 0: the bounds recorded at an epoch, the certificate evaluated after
    # varphi has moved, the sweep's own value beside it.  Entries on the edge of becoming positive, a column that has moved
    # up to 2^12 times as far as everything else is large, every column of the four as the recorded one
    f = np.float32
    fma = lambda a, b, c: (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(f)  # noqa: E731
    fp, up = ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_ubyte)

    def certify(entry, *arrays):
        out = np.zeros(len(arrays[-1]), dtype=np.uint8)
        held = [np.ascontiguousarray(a, dtype=f) if isinstance(a, np.ndarray) else ctypes.c_float(a) for a in arrays]
        entry(len(out), *[a.ctypes.data_as(fp) if isinstance(a, np.ndarray) else a for a in held], out.ctypes.data_as(up))
        return out.astype(bool)

    rng = np.random.default_rng(23)
    N, rho = 400000, f(2.0 / 4000)
    for ratio in (1.0, 4.0, 16.0, 64.0, 4096.0):
        for fallen in (True, False):
            small = f(1.0e-4)
            phi = (small * rng.uniform(-1, 1, N)).astype(f)
            now = (small * rng.uniform(-1, 1, (N, 4))).astype(f)
            then = (now + small * rng.uniform(-1, 1, (N, 4)) * rng.choice([0.0, 1.0], (N, 1))).astype(f)
            big = (ratio * small * rng.uniform(0.5, 1, N)).astype(f)
            then[:, 0] = big if fallen else -big  # the one that moves far
            # the first column (and at random the others) within a few units of the edge, the others well below it
            edge = (now.astype(np.float64) + phi[:, None].astype(np.float64))
            cost = (edge / float(rho) * (1 + rng.uniform(-8, 8, (N, 4)) * 2.0 ** -24)
                    + rng.uniform(-4, 4, (N, 4)) * 2.0 ** -24 * (ratio * float(small)) / float(rho)).astype(f)
            cost[:, 1:] += (rng.choice([0.0, 1.0, 50.0], (N, 3)) * float(small) / float(rho)).astype(f)
            rhos = np.full((N, 4), rho, dtype=f)
            t = fma(-rhos, cost, then)
            order = np.argsort(-t, axis=1, kind="stable")
            star = order[:, 0]
            m1, m2 = np.take_along_axis(t, order[:, :1], 1)[:, 0], np.take_along_axis(t, order[:, 1:2], 1)[:, 0]
            moved = (now - then).astype(f)
            drift1 = np.take_along_axis(moved, star[:, None], 1)[:, 0]
            drift = moved.max(axis=1)
            mag = (np.abs(drift) + np.abs(now).max(axis=1)).astype(f)
            value = fma(-rhos, cost, (now + phi[:, None]).astype(f)).max(axis=1)  # what the sweep clamps
            passed = certify(planlib.drot_certify_segments, m1, m2, drift1, drift, mag, phi)
            assert not (passed & (value > 0)).any(), (ratio, fallen, int((passed & (value > 0)).sum()))
            # the same four as a line of a segment whose largest t lies further up
            top = (m1 + rng.choice([0.0, 0.3, 30.0], N) * float(rho)).astype(f)
            line = certify(planlib.drot_certify_lines, float(rho), top, (top - m1).astype(f), drift, mag, phi)
            assert not (line & (value > 0)).any(), (ratio, fallen, int((line & (value > 0)).sum()))
            # neither is vacuous: a hundred units below the edge almost everything passes
            low = (phi - f(2.0e-4) * f(ratio)).astype(f)
            assert certify(planlib.drot_certify_segments, m1, m2, drift1, drift, mag, low).mean() > 0.5


def test_what_a_list_of_active_entries_leaves_out_stays_zero(planlib):
    # zero entries within a few units in the last place of the edge, with costs that cancel potentials up to 2^20 times as large as what
    # is left: an entry or a line that is not listed stays zero in the sweep behind the list, and in any later one that a rise below the
    # slack leads to, phi and varphi moving as they like
    f = np.float32
    fp, up = ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_ubyte)

    def call(entry, outs, *arrays):
        held = [np.ascontiguousarray(a, dtype=f) for a in arrays]
        entry(len(held[0]), *[a.ctypes.data_as(fp) for a in held], *[o.ctypes.data_as(up if o.dtype == np.uint8 else fp) for o in outs])

    def listed(entry, *arrays):
        out = np.zeros(len(arrays[0]), dtype=np.uint8)
        call(entry, [out], *arrays)
        return out.astype(bool)

    def rises(now, was, other):
        one, both = np.zeros(now.size, dtype=f), np.zeros(now.size, dtype=f)
        call(planlib.drot_active_rises, [one, both], now.ravel(), was.ravel(), other.ravel())
        return one.reshape(now.shape), both.reshape(now.shape)

    # (the sweep clamps fmaf(-rho, c, varphi + phi): its sign is that of the rounded sum less the exact product)
    positive = lambda c, vp, ph: (vp + ph).astype(f).astype(np.float64) > float(rho) * c.astype(np.float64)  # noqa: E731
    rng = np.random.default_rng(29)
    N, rho, small = 200000, f(2.0 / 4000), 1.0e-4
    for ratio in (1.0, 2.0 ** 8, 2.0 ** 14, 2.0 ** 20):
        for slack in (0.0, 1e-3, 1.0):
            phi = (small * rng.uniform(-1, 1, N)).astype(f)
            varphi = (ratio * small * rng.uniform(-1, 1, (N, 4))).astype(f)
            tau = np.full(N, slack * small, dtype=f)
            unit = 2.0 ** -24 * (np.abs(varphi) + np.abs(phi)[:, None] + tau[:, None]).astype(np.float64)
            edge = varphi.astype(np.float64) + phi[:, None] + tau[:, None]
            cost = ((edge + rng.uniform(-24, 48, (N, 4)) * unit) / float(rho)).astype(f)
            t = (-float(rho) * cost.astype(np.float64) + varphi).astype(f)
            # later: they rise and fall by much, together by less than the slack as it is checked
            fall = small * rng.uniform(0, 2, N) * rng.choice([0.0, 1.0], N)
            later_phi = (phi + fall + tau * rng.uniform(-0.5, 1.0, N)).astype(f)
            later = (varphi - fall[:, None]).astype(f)
            up_cols = rises(later, varphi, np.zeros_like(later))[0].max(axis=1)
            lasts = rises(later_phi, phi, up_cols)[1] < tau
            assert slack == 0.0 or ratio > 2.0 ** 8 or lasts.mean() > 0.1
            for e in range(4):
                out = ~listed(planlib.drot_active_entries, t[:, e], varphi[:, e], phi, tau)
                assert not (out & positive(cost[:, e], varphi[:, e], phi)).any(), (ratio, slack)
                assert not (out & lasts & positive(cost[:, e], later[:, e], later_phi)).any(), (ratio, slack)
                assert 0.05 < out.mean() < 0.95  # (neither all nor nothing)
            # the four as a line whose bound is of an earlier varphi, or was made exact after some rise
            earlier = (varphi + ratio * small * rng.uniform(-1, 1, (N, 4)) * rng.choice([0.0, 0.01], (N, 1))).astype(f)
            top = (-float(rho) * cost.astype(np.float64) + earlier).astype(f).max(axis=1)
            rise = rises(varphi, earlier, np.zeros_like(varphi))[0].max(axis=1)
            before = (ratio * small * rng.uniform(-1, 1, N)).astype(f)
            mag = np.abs(varphi).max(axis=1)
            for bound, risen in ((top, rise), ((t.max(axis=1) - before).astype(f), before)):
                out = ~listed(planlib.drot_active_lines, bound, risen, np.abs(risen) + mag, phi, tau)
                for e in range(4):
                    assert not (out & positive(cost[:, e], varphi[:, e], phi)).any(), (ratio, slack)
                    assert not (out & lasts & positive(cost[:, e], later[:, e], later_phi)).any(), (ratio, slack)


def test_the_sweep_by_lines_renews_when_the_rent_has_reached_the_price(planlib):
    def renewals(waste, price, max_since):
        w = np.ascontiguousarray(waste, dtype=np.int32)
        out = np.zeros(len(w), dtype=np.uint8)
        planlib.drot_renewals(len(w), w.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), price, max_since,
                              out.ctypes.data_as(ctypes.POINTER(ctypes.c_ubyte)))
        return np.flatnonzero(out).tolist()

    assert renewals([10] * 40, 100, 1024) == [10, 21, 32]        # ten sweeps' rent, then the one that renews
    assert renewals([10] * 40, 101, 1024) == [11, 23, 35]        # reached, not exceeded
    assert renewals([0] * 40, 100, 5) == [5, 11, 17, 23, 29, 35]  # at the latest after max_since sweeps
    assert renewals([0] * 3000, 100, 1024) == [1024, 2049]
    assert renewals([99, 0, 0, 1, 7, 100, 3], 100, 1024) == [4, 6]  # what the renewing sweep itself reads counts for nothing
    assert renewals([2 ** 31 - 1] * 6, 1000000000, 1024) == [1, 3, 5]  # (lines read in vain beyond the range of the sum)
    # the sum of what was paid since the last renewal, with any rents
    rng = np.random.default_rng(3)
    waste, price = rng.integers(0, 50, 2000), 400
    expect, paid, renew = [], 0, False
    for k, w in enumerate(waste):
        if renew:
            expect.append(k)
            paid, renew = 0, False
        else:
            paid += int(w)
            renew = paid >= price
    assert renewals(waste, price, 1024) == expect


def test_a_stop_at_a_check_forgets_what_the_sweeps_queued_behind_it_would_have_left(planlib):
    # check_every 25, the check at iteration 100 passes; the stretch 101..125 is already queued, and the
    # host-ordered refresh at sweep 122 lies in it: it never runs, so the continued call must not count on it
    t = trace(planlib, 2300, 2500, 5000, reg_kind=1, checking=1, check_every=25, skip_cost=0, screening=1, feedback=1,
              densities=(0.5,), stop_at_status=6)  # statuses: 16, 25, 32, 50, 64, 75, 96?, ...
    ends = [i + 1 for i, f in enumerate(t.col("flags")) if f & 1]
    stop_iter = ends[6]
    assert t.iters == stop_iter and len(t.rows) == ends[7]  # one more stretch was queued
    assert t.carry[2] == -1 and t.carry[3] == 8 and t.carry[4] == 0 and t.carry[6] == 0 and t.carry[7] == stop_iter
    cont = trace(planlib, 2300, 2500, 40, reg_kind=1, checking=1, check_every=25, skip_cost=0, screening=1, resume=1,
                 carry=t.carry, densities=(0.5,))
    assert cont.col("kind")[0] == 6 and cont.col("prev_sums")[0] == 0  # new bounds first, everything read


def test_without_feedback_the_schedule_is_fixed(planlib):
    # (what an entry point that never reads the status block during the solve runs)
    t = trace(planlib, 4096, 4096, 300, reg_kind=1, checking=1, feedback=0, densities=(0.01,))
    assert not t.statics["adaptive"] and t.statics["may_screen"]
    kinds = t.col("kind")
    assert 7 not in kinds and set(t.col("mode")) == {0}
    assert not any(f & 2 for f in t.col("flags"))  # no early looks
    assert [i + 1 for i, f in enumerate(t.col("flags")) if f & 1] == [100, 200, 300]
    assert [i + 1 for i, k in enumerate(kinds) if k == 6] == [2, 10, 26, 58, 122, 250]


def test_gap_checks_ride_on_the_residual_checks(planlib):
    t = trace(planlib, 1000, 1000, 1000, reg_kind=1, checking=1, check_every=100, gap_every=3)
    ends = [(i + 1, bool(f & 4)) for i, f in enumerate(t.col("flags")) if f & 1]
    assert [e for e, g in ends if g] == [300, 600, 900] and len(ends) == 10
    # a gap trace without a tolerance still cuts the solve into stretches
    t = trace(planlib, 1000, 1000, 250, reg_kind=1, checking=0, check_every=100, gap_every=1)
    assert [(i + 1, bool(f & 4)) for i, f in enumerate(t.col("flags")) if f & 1] == [(100, True), (200, True), (250, False)]


def test_point_clouds_and_warm_starts(planlib):
    t = trace(planlib, 3000, 3000, 5, from_points=1, reg_kind=1, checking=0)
    assert set(t.col("sweep")) == {POINTS} and t.col("prev_sums") == [0, 1, 1, 1, 1] and set(t.col("update")) == {MERGED_TILES}
    t = trace(planlib, 3000, 3000, 5, from_points=1, reg_kind=1, checking=0, skip_unchanged=0)
    assert set(t.col("prev_sums")) == {0}
    t = trace(planlib, 2300, 2500, 4, warm=1, reg_kind=1, checking=0, screening=1)
    # the warm start's sums of X_0 serve as flags for the first sweep, which is no "first" sweep (X_0 is read)
    assert t.col("first") == [0, 0, 0, 0] and t.col("prev_sums")[0] == 1 and t.col("kind")[0] == 6
    t = trace(planlib, 5000, 5000, 3, warm=1, reg_kind=2, slab_k=4, nruns=10, checking=0)
    assert t.col("prev_sums") == [0, 1, 1]  # (those sums are per 256 columns, the slab kernel's flags per 32)
    # a warm start with the cost from point clouds: X_0 is read where its sums say so, and the sweep records bounds
    t = trace(planlib, 3000, 3000, 4, from_points=1, warm=1, reg_kind=1, checking=0, screening=1)
    assert set(t.col("sweep")) == {POINTS} and t.col("first") == [0, 0, 0, 0] and t.col("prev_sums") == [1, 1, 1, 1]
    # (the last sweep before a look at the density records the bounds)
    assert t.col("refresh") == [0, 0, 0, 1] and t.col("kind") == [0, 0, 0, 9]


def test_label_analysis(planlib):
    def labels(arr, classes, max_runs=1000, force=0):
        a = np.ascontiguousarray(arr, dtype=np.int32)
        nruns = ctypes.c_int()
        k = planlib.drot_plan_labels(a.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), len(a), classes, max_runs, force,
                                     ctypes.byref(nruns))
        return k, nruns.value

    assert labels(np.repeat(np.arange(10), 500), 10) == (4, 10)       # 500 rows: 4 per row lane
    assert labels(np.repeat(np.arange(3), 128), 3) == (1, 3)
    assert labels(np.repeat(np.arange(2), 1024), 2) == (8, 2)
    assert labels(np.repeat(np.arange(2), 1025), 2) == (0, 2)         # too long for the registers
    assert labels([0, 0, 1, 1, 0], 2) == (0, 3)                       # a class in two runs
    assert labels(np.repeat(np.arange(10), 500), 10, force=1) == (0, 10)
    assert labels(np.repeat(np.arange(10), 5), 10, max_runs=9) == (0, 10)
    assert labels([0, 1, 2, 3], 3)[0] == -1 and labels([0, -1], 3)[0] == -1
    assert labels([2, 2, 2], 5) == (1, 1)                             # unused classes are fine


def test_classes_in_several_runs_are_mapped_to_slabs_where_they_fill_them(planlib):
    ip = ctypes.POINTER(ctypes.c_int)

    def mapped(labels, classes, max_runs=1000, force=0):
        a = np.ascontiguousarray(labels, dtype=np.int32)
        nruns, rows = ctypes.c_int(), np.zeros(8 * 128 * classes, dtype=np.int32)
        k = planlib.drot_plan_labels(a.ctypes.data_as(ip), len(a), classes, max_runs, force, ctypes.byref(nruns))
        got = planlib.drot_plan_label_rows(a.ctypes.data_as(ip), len(a), classes, max_runs, rows.ctypes.data_as(ip), len(rows))
        if k > 0:  # every row of every class that has any, once, in ascending order
            used = [c for c in range(classes) if (a == c).any()]
            table = rows[:got].reshape(len(used), 128 * k)
            for c, r in zip(used, table):
                n = int((a == c).sum())
                assert r[:n].tolist() == np.flatnonzero(a == c).tolist() and (r[n:] == -1).all()
        return k, nruns.value

    rng = np.random.default_rng(11)
    assert mapped(np.arange(256) % 2, 2) == (1, 2) and mapped(np.arange(258) % 2, 2) == (2, 2)
    assert mapped(np.arange(2048) % 2, 2) == (8, 2) and mapped(np.arange(2050) % 2, 2)[0] == 0  # too long for the registers
    assert mapped(rng.permutation(np.arange(2000) % 5), 7) == (4, 5)                            # unused classes
    assert mapped(np.arange(480) % 10, 10) == (1, 10) and mapped(np.arange(479) % 10, 10)[0] == 0  # 3/8 of the row lanes
    assert mapped([0] * 500 + [1] + [0] * 400, 2)[0] == 8 and mapped([0] * 500 + [1, 2, 1] + [0] * 400, 3)[0] == 0
    assert mapped(np.arange(480) % 10, 10, max_runs=9)[0] == 0
    a = np.ascontiguousarray(np.arange(480) % 10, dtype=np.int32)
    assert planlib.drot_plan_labels(a.ctypes.data_as(ip), 480, 10, 1000, 1, ctypes.byref(ctypes.c_int())) == 0
    # consecutive rows need no table
    b = np.repeat(np.arange(3, dtype=np.int32), 100)
    assert planlib.drot_plan_label_rows(b.ctypes.data_as(ip), 300, 3, 1000, None, 0) == 0


def test_the_slabs_fuse_the_update_while_one_round_of_workgroups_holds_them(planlib):
    for n, nruns, small in ((1500, 5, 1), (1500, 6, 0), (2048, 4, 1), (2049, 3, 0), (128, 64, 1), (120, 65, 0)):
        t = trace(planlib, 2000, n, 30, reg_kind=2, slab_k=4, nruns=nruns)
        assert t.statics["small"] == small and set(t.col("sweep")) == {SLAB}
        assert MERGED_SLAB in t.col("update") if not small else MERGED_SLAB not in t.col("update")


def test_class_chunks_of_the_two_pass_group_lasso_path(planlib):
    rng = np.random.default_rng(7)
    for m, classes in ((1, 1), (50, 3), (1000, 7), (333, 40)):
        labels = np.ascontiguousarray(rng.integers(0, classes, size=m), dtype=np.int32)
        if classes > 2:
            labels[labels == 1] = 0  # an empty class
        perm = np.zeros(m, dtype=np.int32)
        cap = m // 16 + classes + 1
        chunk_start = np.zeros(cap + 1, dtype=np.int32)
        class_first = np.zeros(classes + 1, dtype=np.int32)
        ip = ctypes.POINTER(ctypes.c_int)
        nchunks = planlib.drot_plan_chunks(labels.ctypes.data_as(ip), m, classes, perm.ctypes.data_as(ip),
                                           chunk_start.ctypes.data_as(ip), cap, class_first.ctypes.data_as(ip))
        assert nchunks >= 1 and class_first[0] == 0 and class_first[classes] == nchunks and chunk_start[nchunks] == m
        assert sorted(perm.tolist()) == list(range(m))          # a permutation of the rows
        for c in range(classes):
            rows = []
            for k in range(class_first[c], class_first[c + 1]):
                chunk = perm[chunk_start[k]:chunk_start[k + 1]].tolist()
                assert 1 <= len(chunk) <= 16
                rows += chunk
            assert rows == np.flatnonzero(labels == c).tolist()  # every row of the class once, in ascending order


def test_point_cloud_variant_screens_once_the_plan_is_sparse(planlib):
    # looks at 16, 24, 32, ... while the plan is dense, each read at once: 40 % are too many yet, 30 % are not
    t = trace(planlib, 20000, 20000, 200, from_points=1, reg_kind=1, checking=0, densities=(0.9, 0.6, 0.4, 0.3, 0.05))
    kinds = t.col("kind")
    # full sweeps, the last one before a look recording the bounds
    assert kinds[:40] == [0] * 15 + [9] + ([0] * 7 + [9]) * 3
    ends = [i + 1 for i, f in enumerate(t.col("flags")) if f & 1]
    assert ends[:7] == [16, 24, 32, 40, 64, 96, 100]
    # lean from sweep 41, on the bounds of sweep 40; they are renewed by one full sweep after 8 sweeps, then after 16, 32, ...
    assert kinds[40:47] == [8] * 7 and kinds[47] == 9 and kinds[48:63] == [8] * 15 and kinds[63] == 9
    assert t.col("sweep")[40] == POINTS_LEAN and t.col("sweep")[47] == POINTS
    # a plan that stays dense: looks every 8 iterations up to 128, then every 32
    t2 = trace(planlib, 20000, 20000, 240, from_points=1, reg_kind=1, checking=0, densities=(0.9,))
    ends = [i + 1 for i, f in enumerate(t2.col("flags")) if f & 1]
    assert ends == sorted({16, 100, 200, 240} | set(range(24, 129, 8)) | {160, 192, 224}) and 8 not in t2.col("kind")
    assert [k == 9 for k in t2.col("kind")] == [i + 1 in ends for i in range(240)]
    # column sums: eight 32-row tiles of the full sweep are added first, as the strips of the screened sweep store them
    assert t.col("ra")[5] == 625 * 16 + 8 and t.col("ra")[41] == 79 * 16 + 1 and t.col("ra")[0] == 625 * 16 + 8
    # one launch for the vector update: the sweeps store the totals of their tiles (the screened one of its strips)
    assert set(t.col("update")) == {MERGED_TILES} and set(t.col("tilesum")) == {1}
    # small problems, or with the screening off: the full sweep only, column sums ungrouped
    t = trace(planlib, 3000, 3000, 40, from_points=1, reg_kind=1, checking=0, densities=(0.05,))
    assert set(t.col("kind")) == {0} and set(t.col("ra")) == {94 * 16 + 8}
    t = trace(planlib, 20000, 20000, 120, from_points=1, reg_kind=1, checking=0, screening=0, densities=(0.05,))
    assert set(t.col("kind")) == {0}
    # a warm start looks as early as a cold one; a continued call not at all before its checks, and records before them
    t = trace(planlib, 20000, 20000, 60, from_points=1, warm=1, reg_kind=1, checking=0, densities=(0.3,))
    assert t.col("kind")[:17] == [0] * 15 + [9, 8]
    t = trace(planlib, 20000, 20000, 250, from_points=1, reg_kind=1, checking=1, resume=1, densities=(0.3,),
              carry=(0, -1000000, -1, 8, 1, 256, 0, 100))
    assert t.col("kind") == ([0] * 99 + [9]) * 2 + [8] * 7 + [9] + [8] * 15 + [9] + [8] * 26
    # a continued call goes on with the bounds it finds
    first = trace(planlib, 20000, 20000, 100, from_points=1, reg_kind=1, checking=0, densities=(0.9, 0.6, 0.2, 0.05))
    cont = trace(planlib, 20000, 20000, 20, from_points=1, reg_kind=1, checking=0, resume=1, carry=first.carry, densities=(0.05,))
    assert cont.col("kind")[0] == 8


def test_grid_resident_stretches_where_the_registers_of_the_chip_hold_the_problem(planlib):
    def grid(m, n, iters=300, units=256, single=0, reg_kind=1, from_points=0, warm=0, feedback=1, slab_k=0, nruns=0,
             check_every=100, fused_update=-1, skip_cost=-1, skip_unchanged=-1, screening=-1):
        problem = (ctypes.c_int * 14)(m, n, reg_kind, from_points, warm, 0, 0, 1, 1, slab_k, nruns, feedback, 1, iters)
        options = (ctypes.c_int * 9)(check_every, -1, fused_update, skip_cost, skip_unchanged, screening, -1, 0, 0)
        out = (ctypes.c_int * 4)()
        planlib.drot_plan_grid(problem, options, units, single, out)
        return tuple(out)

    assert grid(100, 100)[0] == 0                                  # one workgroup does it
    assert grid(129, 2)[:3] == (1, 32, 0)
    assert grid(1000, 1000) == (1, 32, 0, 0)
    assert grid(2048, 1024 * 5)[:2] == (5, 32) and grid(2048, 1024 * 5 + 1)[0] == 0   # 64 rows of tiles x 20, x 21 columns
    # beyond the fused path: 64-row tiles; the first sweep of a cold start goes by itself, a warm start has no such
    assert grid(2999, 3307)[:3] == (3, 64, 1) and grid(2999, 3307, warm=1)[2] == 0
    assert grid(3072, 4096, screening=0)[0] == 3 and grid(3073, 4096, screening=0)[0] == 0 and grid(3072, 4096)[0] == 0
    assert grid(2999, 3307, screening=1)[0] == 0 and grid(2999, 3307, skip_cost=1)[0] == 0
    assert grid(2999, 3307, skip_unchanged=0)[0] == 0 and grid(1000, 1000, fused_update=0)[0] == 0
    # every row and column needs a wave to form its part of eq. (6), eight to a wave
    assert grid(32, 5000)[:2] == (1, 32) and grid(2, 65000)[0] == 0
    # short stretches and callers that want every sweep in a launch of its own
    assert grid(1000, 1000, check_every=3)[2] == -1 and grid(1000, 1000, iters=3)[2] == -1
    assert grid(1000, 1000, iters=7)[2] == -1 and grid(1000, 1000, iters=8)[2] == 0          # one tile a workgroup: 8 sweeps
    assert grid(2048, 3072, iters=3)[2] == -1 and grid(2048, 3072, iters=4)[2] == 0          # more tiles, or 64-row tiles: 4
    assert grid(2999, 3307, iters=4)[2] == -1 and grid(2999, 3307, iters=5)[2] == 1 and grid(2049, 256, iters=5)[2] == 1
    assert grid(1000, 1000, single=1)[2] == -1 and grid(1000, 1000, units=0)[0] == 0
    assert grid(1000, 1000, units=32)[0] == 4 and grid(2048, 2048, units=32)[0] == 0  # a smaller partition of the chip
    assert grid(1000, 1000, from_points=1)[0] == 0 and grid(1000, 1000, reg_kind=2)[0] == 0
    # no even/odd pairs where nothing is streamed, whoever asks for single launches
    assert grid(2999, 3307)[3] == 0 and grid(2999, 3307, single=1)[3] == 0 and grid(2999, 3307, units=0)[3] == 1


def test_launches_run_on_through_the_residual_checks(planlib):
    def run(m, n, iters, check_every=100, k=0, feedback=1, checking=1, resident=-1, gap_every=0, units=256, single=0, from_points=0,
            skip_unchanged=-1, screening=-1):
        problem = (ctypes.c_int * 14)(m, n, 1, from_points, 0, 0, 0, 1, 1, 0, 0, feedback, checking, iters)
        options = (ctypes.c_int * 9)(check_every, resident, -1, -1, skip_unchanged, screening, -1, 0, gap_every)
        return planlib.drot_plan_run(problem, options, units, single, k)

    for m, n in ((100, 100), (1000, 1000), (2999, 3307)):
        assert run(m, n, 1000) == 1000 and run(m, n, 130) == 130 and run(m, n, 130, k=70) == 60 and run(m, n, 7, check_every=1) == 7
        # the host looks at them after 4096 sweeps or 256 checks, at a check each time
        assert run(m, n, 100000) == 4000 and run(m, n, 100000, k=150) == 50 + 4000 and run(m, n, 1000, check_every=1) == 256
        assert run(m, n, 100000, check_every=5000) == 5000 and run(m, n, 6000, check_every=5000, k=5000) == 1000
        # not where the gap is evaluated at checks, nothing is tested, the host reads no status, or every sweep is timed
        assert run(m, n, 1000, gap_every=1) == 0 and run(m, n, 1000, checking=0) == 0 and run(m, n, 1000, feedback=0) == 0
        assert run(m, n, 1000, single=1) == 0
    assert run(100, 100, 1000, units=0) == 1000 and run(1000, 1000, 1000, units=0) == 0 and run(5000, 5000, 1000) == 0
    # point clouds: up to five 32-row tiles per workgroup, whatever the rows; not where screened or told to move every byte
    assert run(100, 100, 1000, from_points=1) == 1000 and run(3200, 3072, 1000, from_points=1) == 1000
    assert run(3200, 3328, 1000, from_points=1) == 0 and run(5000, 5000, 1000, from_points=1) == 0
    assert run(1000, 1000, 1000, from_points=1, screening=1) == 0 and run(1000, 1000, 1000, from_points=1, skip_unchanged=0) == 0
    assert run(2, 32600, 1000) == 1000 and run(2, 32640, 1000) == 0  # (more blocks of columns than workgroups own)


def test_grid_resident_slabs_where_every_workgroup_holds_one(planlib):
    def slabs(m, n, k, nruns, mapped=0, fused_update=-1, units=256):
        out = (ctypes.c_int * 4)()
        planlib.drot_plan_slabs(m, n, k, nruns, mapped, fused_update, units, out)
        return tuple(out)

    assert slabs(1500, 1000, 8, 2) == (1, 4, 8, 128) == slabs(1500, 1000, 8, 2, mapped=1)     # half slabs
    assert slabs(150, 300, 1, 2) == (1, 4, 4, 40)                                             # idle rows
    assert slabs(2048, 2048, 8, 2) == (1, 4, 8, 256) and slabs(2048, 2049, 8, 2) == (1, 8, 8, 130)
    assert slabs(2000, 1500, 4, 5) == (1, 8, 4, 235) and slabs(1024, 8192, 8, 1) == (1, 8, 8, 256)
    assert slabs(2000, 2500, 4, 5) == (2, 8, 4, 198) and slabs(2048, 4096, 4, 4) == (2, 8, 4, 256)
    assert slabs(2048, 4097, 4, 4)[0] == 0 and slabs(1024, 8193, 8, 1)[0] == 0 and slabs(5000, 5000, 4, 10)[0] == 0
    # no workgroup without a slab: their waves own the blocks of eight rows and columns
    assert slabs(700, 90, 8, 1)[0] == 0 and slabs(1024, 256, 8, 1)[0] == 0 and slabs(1024, 384, 8, 1) == (1, 4, 8, 24)
    # not beside the separate vector update it is compared with, nor without cooperative launches; a smaller partition
    assert slabs(1500, 1000, 8, 2, fused_update=0)[0] == 0 and slabs(1500, 1000, 8, 2, units=0)[0] == 0
    assert slabs(1500, 1000, 8, 2, units=64) == (1, 8, 8, 64) and slabs(1500, 1000, 8, 2, units=32)[0] == 0


def test_separate_vector_updates_keep_point_clouds_and_slabs_off_the_cooperative_launches(planlib):
    # the option says so: a launch for every sweep
    out = (ctypes.c_int * 4)()
    for m, n, k, nruns, mapped in ((1500, 1000, 8, 2, 0), (1000, 3001, 8, 1, 0), (2000, 2500, 4, 5, 0), (2000, 1500, 4, 5, 1), (1024, 8192, 8, 1, 1)):
        for fused, held in ((-1, True), (0, False)):
            planlib.drot_plan_slabs(m, n, k, nruns, mapped, fused, 256, out)
            assert (out[0] > 0) == held, (m, n, fused)
    for m, n in ((100, 100), (1000, 1000), (3200, 3072)):
        problem = (ctypes.c_int * 14)(m, n, 1, 1, 0, 0, 0, 1, 1, 0, 0, 1, 1, 1000)
        for fused, sweeps in ((-1, 1000), (0, 0)):
            options = (ctypes.c_int * 9)(100, -1, fused, -1, -1, -1, -1, 0, 0)
            assert planlib.drot_plan_run(problem, options, 256, 0, 0) == sweeps, (m, n, fused)


def test_launches_of_calls_without_checks_are_bounded_where_sweeps_were_launches(planlib):
    # point clouds and slabs; stored costs on tiles have always run such a call in one launch
    def stretch(m, n, iters, k=0, reg_kind=1, from_points=0, slab_k=0, nruns=0, checking=0, units=256, fused_update=-1, check_every=100):
        problem = (ctypes.c_int * 14)(m, n, reg_kind, from_points, 0, 0, 0, 1, 1, slab_k, nruns, 1, checking, iters)
        return planlib.drot_plan_stretch(problem, (ctypes.c_int * 9)(check_every, -1, fused_update, -1, -1, -1, -1, 0, 0), units, k)

    for kw in (dict(from_points=1), dict(reg_kind=2, slab_k=8, nruns=2)):
        assert stretch(1500, 1000, 100000, **kw) == 4096 and stretch(1500, 1000, 100000, k=98304, **kw) == 1696
        assert stretch(1500, 1000, 4096, **kw) == 4096 and stretch(1500, 1000, 500, **kw) == 500
        assert stretch(1500, 1000, 100000, checking=1, **kw) == 100 and stretch(1500, 1000, 100000, checking=1, check_every=5000, **kw) == 5000
        # (single launches need no bound)
        assert stretch(1500, 1000, 100000, units=0, **kw) == 100000 and stretch(1500, 1000, 100000, fused_update=0, **kw) == 100000
    assert stretch(1500, 1000, 100000) == 100000


def _active(planlib, m, n, k=32, iters=1000, density=0.3, lines=0.03, by_lines=1, epoch=8, left=0, ago=0, before=0.3, forecast=-1.0, units=256, single=0, reg_kind=1,
            from_points=0, feedback=1, check_every=100, fused_update=-1, skip_cost=-1, skip_unchanged=-1, screening=-1, gap_every=0):
    problem = (ctypes.c_int * 14)(m, n, reg_kind, from_points, 0, 0, 0, 1, 1, 0, 0, feedback, 1, iters)
    options = (ctypes.c_int * 9)(check_every, -1, fused_update, skip_cost, skip_unchanged, screening, -1, 0, gap_every)
    state = (ctypes.c_int * 9)(k, int(density * 1e6), int(lines * 1e6), by_lines, epoch, left, ago, int(before * 1e6), int(forecast * 1e6))
    out = (ctypes.c_int * 8)()
    ever = planlib.drot_plan_active(problem, options, units, single, state, out)
    return ever, tuple(out)


def test_active_entries_of_point_clouds_that_did_not_fit(planlib):
    def active(m=5000, n=4000, **kw):
        return _active(planlib, m, n, from_points=1, lines=-1.0, **kw)[1]

    # tried again early where the plan has thinned out since, and else like any other
    assert active(k=40, left=1, ago=8, density=0.3, before=0.5)[0] > 0 and active(k=40, left=1, ago=7, density=0.3, before=0.5)[0] == 0
    assert active(k=40, left=1, ago=8, density=0.41, before=0.5)[0] == 0 and active(k=40, left=2, ago=15, density=0.1, before=0.5)[0] == 0
    assert active(k=700, left=1, ago=511, density=0.1, before=0.5)[0] == 0 and active(k=700, left=1, ago=512, density=0.5, before=0.3)[0] > 0
    # what was known of the plan before such a launch is not known of it behind it, and the host waits for the next look
    assert active(k=40)[3:5] == (-1, 1)
    assert _active(planlib, 10000, 10000)[1][3:5] == (300000, 0)
    # a list has to last the longer, the less a sweep over everything takes
    assert active(2500, 15360, k=16)[5] == 6 and active(2499, 15360, k=16)[5] == 10 and active(20000, 20000, k=16)[5] == 6
    assert _active(planlib, 10000, 10000)[1][5] == 16


def test_active_entries_counted_in_advance(planlib):
    def active(forecast, lines=0.1, **kw):  # (10000 x 10000: lines of 0.1, 0.15 and 0.19 are 0.47, 0.73 and 0.95 of the room)
        return _active(planlib, 10000, 10000, lines=lines, forecast=forecast, **kw)[1]

    # where such a launch may come, over a stored cost, and bounds are there to count by
    assert active(-1.0)[6] == 1 and active(-1.0, lines=0.5)[6] == 1
    for other in (dict(by_lines=0), dict(epoch=-1), dict(iters=47), dict(left=1, ago=511, k=600), dict(units=255), dict(from_points=1), dict(single=1)):
        assert active(-1.0, **other)[6] == 0, other
    # the count decides: more of it in the first iterations, whose rise does not last, and where the plan alone has little; never past what the
    # plan alone would take
    assert active(0.93, lines=0.15)[0] > 0 and active(0.95, lines=0.15)[0] == 0 and active(0.93, lines=0.19)[0] > 0 and active(0.93, lines=0.21)[0] == 0
    assert active(1.11)[0] > 0 and active(1.13)[0] == 0
    assert active(1.19, k=16)[0] > 0 and active(1.21, k=16)[0] == 0 and active(1.19, k=16, lines=0.21)[0] == 0
    # what lies within the slack does not go away: the host neither waits for the looks that follow nor tries before 512 iterations are over; a plan
    # that is still thinning is looked at again
    assert active(1.13, lines=0.095)[:2] == (0, 32 + 512) and active(1.13, lines=0.095)[4] == 0
    assert active(0.95, lines=0.15)[:2] == (0, 42 + 512)


def test_active_entries_once_a_large_plan_is_known_to_be_thin(planlib):
    def active(*args, **kw):
        ever, out = _active(planlib, *args, **kw)
        return ever, out[:3]

    # runs on through the checks, 2048 iterations (point clouds: 1024) or 256 checks at a time
    assert active(10000, 10000) == (1, (968, 42 + 512, 1))
    assert active(10000, 10000, iters=100000)[1][0] == 68 + 1900 and active(10000, 10000, iters=2032 + 48)[1][0] == 2048
    assert active(12000, 12000, iters=100000, from_points=1)[1][0] == 68 + 900
    assert active(10000, 10000, iters=100000, check_every=5000)[1][0] == 4968  # (or to one check)
    assert active(10000, 10000, k=30, iters=1000, check_every=1)[1][0] == 256
    # sizes: 80 segments of 256 columns and groups of 256 rows at most, 11.5 million entries at least
    assert active(20480, 20480)[0] == 1 and active(20481, 1000)[0] == 0 and active(1000, 20481)[0] == 0
    assert active(3396, 3397)[0] == 1 and active(3396, 3396)[0] == 0 and active(2049, 20480)[0] == 1 and active(600, 20480, from_points=1)[0] == 1
    assert active(2048, 16384)[0] == 0 and active(2049, 16384)[0] == 1  # (few enough rows for the vector update to ride on the sweep)
    # who asks for something else, or where the host does not look
    for other in (dict(units=255), dict(fused_update=0), dict(skip_cost=1), dict(skip_unchanged=0), dict(screening=0), dict(screening=1),
                  dict(gap_every=1), dict(feedback=0), dict(reg_kind=2)):
        assert active(10000, 10000, **other) == (0, (0, 42 + 512, 1)), other
    assert active(10000, 10000, single=1)[1][0] == 0
    # not before the plan is known to be thin (0.75 of the room for entries of the workgroup that has most rows and columns, each entry by its
    # own chance), nor without bounds, nor for the last few
    for m, n in ((10000, 10000), (20000, 20000), (4000, 4000), (4200, 12290), (5000, 5000)):
        most = [max(sum(min(256, k - at) for at in range(256 * w, k, 4096)) for w in range(16) if 256 * w < k) for k in (m, n)]
        share = 0.75 * 4096 / (most[0] * most[1])
        lines = 1.0 - (1.0 - share) ** 32
        assert active(m, n, lines=0.99 * lines)[1][0] > 0 and active(m, n, lines=1.01 * lines)[1][0] == 0
        assert abs(_active(planlib, m, n, lines=lines)[1][7] - 750000) < 200
        assert active(m, n, lines=-1.0)[1][0] == 0 and active(m, n, by_lines=0)[1][0] == 0 and active(m, n, epoch=-1)[1][0] == 0
        assert active(m, n, iters=48)[1][0] == 16 and active(m, n, iters=47)[1][0] == 0
        assert active(m, n, from_points=1, lines=-1.0, by_lines=0)[1][0] > 0
        assert active(m, n, from_points=1, density=0.61)[1][0] == 0 and active(m, n, from_points=1, density=-1.0)[1][0] == 0
    assert active(12000, 12000, from_points=1, density=0.59)[1][0] > 0
    # one that ended early is not tried again at once, and later every time
    assert active(12000, 12000, k=16, from_points=1)[1][1] == 26 + 8
    assert active(10000, 10000, k=200, left=1, ago=511)[1][0] == 0 and active(10000, 10000, k=200, left=1, ago=512)[1] == (800, 210 + 1024, 2)
    assert active(10000, 10000, k=900, left=3, ago=2047)[1][0] == 0 and active(10000, 10000, k=900, left=3, ago=2048)[1][0] == 100


# calls of one handle, each continuing the last: what the options of a call leave out (the defaults of a case are those of the first)
@pytest.mark.parametrize("from_points", [1, 0])
@pytest.mark.parametrize("off", [dict(gap_every=1), dict(fused_update=0), dict(screening=1)])
@pytest.mark.parametrize("order", [(0, 1), (1, 0, 1), (1, 0, 0, 1), (0, 1, 0, 1)])
def test_active_entries_start_from_bounds_that_are_there(planlib, from_points, off, order):
    calls = []
    for on in order:
        o = dict(check_every=20, fused_update=-1, screening=-1, gap_every=0)
        o.update({} if on else off)
        calls += [o["check_every"], -1, o["fused_update"], 0, -1, o["screening"], -1, 0, o["gap_every"]]
    problem = (ctypes.c_int * 14)(6000, 6000, 1, from_points, 0, 0, 0, 1, 1, 0, 0, 1, 1, 0)
    events = (ctypes.c_longlong * 4000)()
    count = planlib.drot_plan_active_calls(problem, len(order), (ctypes.c_int * len(calls))(*calls),
                                           (ctypes.c_int * len(order))(*([300, 240, 180, 200][:len(order)])), 256, 200000, 20000, events, 1000)
    assert 0 < count <= 1000
    # what is in memory: the iteration whose varphi the bounds by line are against, that of the last epoch's varphi and that of the
    # varphi a launch left with its bounds
    bounds = epoch = left = None
    launches = 0
    for e in range(count):
        launch, a, b, source = events[4 * e:4 * e + 4]
        if not launch:
            epoch = a
            if b:
                bounds = a
        else:
            launches += 1
            against = {1: left, 2: epoch}[source]
            assert bounds is not None and against == bounds, (e, a, source)
            bounds = left = b
    # ... and every call at the defaults takes such launches, the first one of a continued call as soon as there are bounds
    assert launches >= sum(order)
