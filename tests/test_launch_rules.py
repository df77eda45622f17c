"""The launch rules (csrc/launch_rules.h), built with plain g++ and asked for their answers.  No GPU involved."""
import ctypes
import math
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
UNITS = 256


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    lib = tmp_path_factory.mktemp("rules") / "rules.so"
    csrc = os.path.join(ROOT, "paper_2205_00119_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", f"-I{csrc}", "-o", str(lib),
                    os.path.join(ROOT, "tests", "host", "launch_rules_c.cpp")], check=True)
    lib = ctypes.CDLL(str(lib))
    lib.rules_lds.restype = ctypes.c_size_t
    lib.rules_lds.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_size_t]
    lib.rules_copies.restype = ctypes.c_longlong
    lib.rules_copies.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t]
    lib.rules_unrolled.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t]
    lib.rules_shallow.restype = ctypes.c_longlong
    lib.rules_shallow.argtypes = [ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t]
    lib.rules_shallow_segments.restype = ctypes.c_longlong
    lib.rules_shallow_segments.argtypes = [ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t, ctypes.c_size_t]
    lib.rules_segments.restype = ctypes.c_longlong
    lib.rules_segments.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_size_t]
    lib.rules_in_step.argtypes = [ctypes.POINTER(ctypes.c_size_t), ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t]
    lib.rules_reduce.restype = ctypes.c_longlong
    lib.rules_reduce.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_int, ctypes.c_size_t]
    lib.rules_shallow_call.argtypes = [ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t]
    return lib


PIECE, PIECES, MOST = 1280, 128, 65536       # LDS is handed out in pieces, 160 KiB of it a compute unit, 64 KiB a workgroup


HAD = sorted({PIECES // m for m in range(1, MOST // PIECE + 1)})         # numbers of workgroups that a request can leave room for


def workgroups(lds):
    return PIECES // -(-lds // PIECE) if lds else 1 << 20


@pytest.mark.parametrize("lanes", [64, 128, 136, 200, 256, 264, 384, 448, 512])
def test_a_cap_on_wavefronts_is_one(rules, lanes):
    """The dynamic LDS of a workgroup lets no more wavefronts on a compute unit than asked for (but one workgroup, and two where
    64 KiB a workgroup allow no less), and no fewer than can be had."""
    of_one = -(-lanes // 64)                 # a last wavefront that is a partial one counts
    for cap in range(1, 32):
        if cap // of_one >= 32:
            continue
        lds = rules.rules_lds(lanes, cap, 0)
        assert lds <= MOST
        at_most = [c for c in HAD if c <= max(cap // of_one, 1)]
        assert workgroups(lds) == (max(at_most) if at_most else min(HAD)), (cap, lds)
    assert rules.rules_lds(lanes, 0, 0) == 0 and rules.rules_lds(lanes, 0, 4096) == 4096
    assert rules.rules_lds(lanes, 32, 20000) >= 20000


def test_caps_that_can_be_had_exactly(rules):
    assert [c for c in HAD if c < 32] == [2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 14, 16, 18, 21, 25]


def shape(code):
    return code // 64, code % 64


@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("mb", [3, 8, 14, 20, 30, 40, 50, 120, 150, 180, 220, 250, 290, 320, 500, 900, 2000])
def test_no_number_of_copies_stands_alone(rules, fused, mb):
    """From 9 copies on a call of some size is launched as those of one copy less or one more are."""
    def answer(r):
        count = mb * 10**6 // (4 * r + (26 if fused else 4))
        lanes, cap = shape(rules.rules_copies(fused, r, count, UNITS))
        # how many lanes a small call takes follows its elements, not its copies
        return rules.rules_unrolled(fused, r, count, UNITS), (lanes, cap) if mb >= 220 else cap
    answers = {r: answer(r) for r in range(9, 65)}
    for r in range(10, 64):
        assert answers[r] in (answers[r - 1], answers[r + 1]), (r, answers[r - 1], answers[r], answers[r + 1])


@pytest.mark.parametrize("r", [9, 11, 12, 13, 16, 24, 64])
def test_averages_of_many_copies_stay_with_full_size_workgroups_that_run_at_once(rules, r):
    """60 to 96 MiB: up to 24 wavefronts a unit are three full-size workgroups, and from 32 on their number hardly matters."""
    for mib in (61, 66, 72, 80, 88, 95):
        count = mib * 2**20 // (4 * r + 4)
        waves = count // 4 // (64 * UNITS)
        lanes, cap = shape(rules.rules_copies(0, r, count, UNITS))
        if 25 <= waves < 32:
            assert lanes == 64 and cap > 0, (mib, lanes, cap)
        else:
            assert cap == 0, (mib, lanes, cap)


@pytest.mark.parametrize("r", range(1, 9))
def test_updates_go_to_single_wavefronts_where_full_size_workgroups_no_longer_run_at_once(rules, r):
    """From 76 MiB on, but up to 8 copies not below 25 wavefronts a unit."""
    for mib in (40, 60, 75, 77, 80, 83, 88, 92, 100):
        count = mib * 2**20 // (4 * r + 26)
        single = mib > 76 and count // 4 >= 1600 * UNITS
        assert (shape(rules.rules_copies(1, r, count, UNITS))[1] > 0) == single, mib
        if r in (3, 5, 6, 7):
            assert rules.rules_unrolled(1, r, count, UNITS) == single, mib


@pytest.mark.parametrize("r", [6, 7, 9, 12, 13, 14, 16])
def test_averages_keep_the_kernel_for_any_number_of_copies_in_the_middle(rules, r):
    """Unrolled up to one full-size workgroup a unit and, but for 14 and more copies, in large calls."""
    one = 512 * 4 * UNITS
    large = ((60 if r < 8 else 200) << 20) // (4 * r + 4) + 1
    for count, unrolled in ((5, 1), (one, 1), (one + 1, 0), (large - 2, 0), (large, r < 14)):
        assert rules.rules_unrolled(0, r, count, UNITS) == unrolled, count


@pytest.mark.parametrize("p", [16, 19, 20, 24, 31, 32, 48, 64, 96, 128])
def test_shallow_batches_leave_no_round_of_wavefronts_nearly_empty(rules, p):
    """At every size the cap is one of those measured, and the last round is at least four fifths full on its share of the call."""
    for quarter in range(4 * 7, 4 * 400):
        lanes, cap = shape(rules.rules_shallow(p, quarter * 16 * UNITS, UNITS))
        rounds = quarter / 4 / cap if cap else 0
        assert lanes == 64 and cap in (6, 7, 8, 9, 10, 11, 12, 14, 16), (quarter / 4, cap)
        assert rounds <= 1 or rounds / math.ceil(rounds) > .84, (quarter / 4, cap)


@pytest.mark.parametrize("p,per_unit,cap", [(64, 118, 7), (64, 144.5, 7), (96, 68.7, 7), (64, 72.2, 7), (96, 57.2, 6), (96, 95.4, 6), (64, 39.3, 8), (48, 110, 8), (16, 384, 8)])
def test_shallow_batches_of_long_calls(rules, p, per_unit, cap):
    assert shape(rules.rules_shallow(p, int(per_unit * 64) * UNITS, UNITS)) == (64, cap)


@pytest.mark.parametrize("p,per_unit,n,lanes", [
    (64, 5.6, 16, 512), (64, 5.6, 2, 512), (48, 7.7, 16, 512), (128, 7, 16, 512), (64, 15, 16, 512), (96, 23, 16, 512), (64, 8.5, 16, 64), (64, 12.5, 16, 64), (64, 17, 16, 64),
    (64, 15, 4, 64), (128, 26, 16, 64), (64, 30, 16, 64), (47, 7, 16, 64), (64, 7.9, 40, 64), (64, 7.6, 30, 256), (64, 11.5, 16, 256), (64, 11.5, 8, 64),
    (64, 19, 16, 256)])
def test_segments_in_shallow_batches_fill_the_units_evenly(rules, p, per_unit, n, lanes):
    """From 48 buffers on, full-size workgroups where a unit gets one, or a call of many segments two or three, nearly filled, and
    workgroups of 256 lanes for two, three or five; 40 segments of 7.9 wavefronts a unit are more of them than two."""
    assert shape(rules.rules_shallow_segments(p, int(per_unit * 64 * UNITS / n), n, UNITS))[0] == lanes


@pytest.mark.parametrize("p", [1, 2, 3])
def test_segments_of_few_f32_buffers(rules, p):
    for per_unit, lanes in ((20, 256), (49, 256), (50, 64), (100, 64), (299, 64), (600, 64)):
        for accumulate in (0, 1):
            assert shape(rules.rules_segments(p, 4, per_unit * 64 * UNITS, 16, accumulate, UNITS)) == (lanes, 0), per_unit


def test_buffers_in_step(rules):
    """16 MiB from one to the next, up or down, up to 63 of them also 32, in calls of 46 wavefronts a unit."""
    def answer(p, mib, per_unit=58, moved=0):
        at = [(1 << 40) + 12345 * 64 + int(q * mib * 2**20) for q in range(p)]
        at[p // 2] += moved
        return rules.rules_in_step((ctypes.c_size_t * p)(*at), p, per_unit * 64 * UNITS, UNITS)
    for p in (32, 33, 63, 64, 96, 128):
        assert answer(p, 16) and answer(p, -16)
        assert bool(answer(p, 32)) == (p < 64) and bool(answer(p, -32)) == (p < 64)
        assert not answer(p, 16, per_unit=45) and not answer(p, 16, moved=2) and not answer(p, 16, moved=2**21)
        assert not any(answer(p, mib) for mib in (0, 4, 8, 14, 20, 24, 48, 64))
    assert not answer(31, 16) and not answer(16, 16)


def test_partial_last_wavefronts_only_in_kernels_that_know_them(rules):
    """Kernels that pass their stores through LDS: two-byte gradients, accumulator not left in the L2."""
    seen = 0
    for p in range(1, 129):
        for nlanes in range(100, 512 * UNITS, 997):
            for units in (UNITS, 104):
                lanes = shape(rules.rules_reduce(p, 2, nlanes, 0, units))[0]
                assert lanes % 8 == 0 and (lanes % 64 == 0 or rules.rules_partial_waves(p)), (p, nlanes, lanes)
                seen += lanes % 64 != 0
    assert seen > 1000


def test_one_full_size_workgroup_for_every_unit_is_not_read_in_shallow_batches_by_32_buffers(rules):
    """A power of two for counts that are: 64 MB messages over 32 ranks."""
    one = 512 * UNITS
    for p, at, above in ((15, 0, 0), (16, 1, 1), (31, 1, 1), (32, 0, 1), (39, 0, 1), (40, 1, 1), (64, 1, 1)):
        assert bool(rules.rules_shallow_call(p, one, UNITS)) == bool(at) and bool(rules.rules_shallow_call(p, one + 1, UNITS)) == bool(above), p
