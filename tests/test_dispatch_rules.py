"""The dispatch's choices by size alone (csrc/rules.h), compiled for the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_16786_amd", "csrc")

_WRAPPERS = """
#include "rules.h"
extern "C" {
int round_units(int units, int most, int windows) { return fc::round_units(units, most, windows); }
long long residual_cost(int units, int windows) { return fc::residual_cost(units, windows); }
unsigned long long grid_start(unsigned long long at) { return fc::grid_start(at); }
unsigned long long grid_slack() { return fc::kGridSlack; }
int xcd_items(int along, int first, int second) { return fc::xcd_items(along, {first, second}); }
int xcds_along(int f1, int s1, int f2, int s2) { return fc::xcds_along({f1, s1}, {f2, s2}, 0); }
int xcds_along_at_once(int f1, int s1, int f2, int s2, int at_once) { return fc::xcds_along({f1, s1}, {f2, s2}, at_once); }
void xcd_rectangle(int xcd, int along, int first, int second, int* out) {
  const fc::Span a = fc::xcd_first(xcd, along, first), b = fc::xcd_second(xcd, along, second);
  out[0] = a.from; out[1] = a.count; out[2] = b.from; out[3] = b.count;
}
int slot_waves(int slots) { return fc::slot_waves(slots); }
int lane_slot(int part, int lane, int slots) { return fc::lane_slot(part, lane, slots); }
bool round_keeps_rows(long long bytes, int row_bytes) { return fc::round_keeps_rows(bytes, row_bytes); }
void residual_plan(int wins, int tpw, int slots, int units, int f, int sec, bool bf16, int* out) {
  const fc::ResidualPlan p = fc::residual_plan(wins, tpw, slots, units, {f, sec}, bf16);
  out[0] = p.waves; out[1] = p.abreast; out[2] = p.blocks; out[3] = p.split; out[4] = p.once; out[5] = p.along; out[6] = p.workgroups;
}
int residual_groups(bool bf16, bool once, int waves, int slots) { return fc::residual_groups(bf16, once, waves, slots); }
int decimate_tiles(int m, int groups, int steps, bool bf16, int slots, long long row_bytes) {
  return fc::decimate_tiles(m, groups, steps, bf16, slots, row_bytes);
}
int copy_groups(int lists, int layers, int n, int heads, long long rows, int vec_per_row, bool paged) {
  return fc::copy_groups(lists, layers, n, heads, rows, vec_per_row, paged);
}
bool pads_apart(int radix, int done, int group) { return fc::pads_apart(radix, done, group); }
bool keeps_rows(long long rows, int row_bytes) { return fc::keeps_rows(rows, row_bytes); }
bool ranks_by_budget(long long rows, int layers, int splits, int row_bytes) { return fc::ranks_by_budget(rows, layers, splits, row_bytes); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    where = tmp_path_factory.mktemp("rules")
    src, lib = str(where / "rules.cpp"), str(where / "rules.so")
    with open(src, "w") as f:
        f.write(_WRAPPERS)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, src, "-o", lib], check=True)
    return ctypes.CDLL(lib)


def test_rounds_are_as_few_as_whole_sets_allow_and_end_with_the_workgroups_turns(rules):
    rules.residual_cost.restype, rules.residual_cost.argtypes = ctypes.c_longlong, [ctypes.c_int, ctypes.c_int]
    cost = rules.residual_cost
    assert [cost(u, 22) for u in (4, 8, 40, 44, 52, 56, 64)] == [1 * 32, 2 * 33, 7 * 32, 8 * 33, 9 * 32, 10 * 33, 11 * 32]
    for windows in (1, 5, 22, 86, 1024):
        for most in list(range(1, 90)) + [200, 480, 1000]:
            for units in list(range(1, 260)) + [896, 4000, 32767]:
                got = rules.round_units(units, most, windows)
                if units <= most or most < 4:
                    assert got == min(units, most)
                    continue
                cap = most // 4 * 4
                rounds = -(-units // cap)
                assert 4 <= got <= cap and got % 4 == 0, (units, most, windows, got)
                assert -(-units // got) == rounds, (units, most, windows, got)       # (no round for what is left over)

                def of(c):
                    return sum(cost(min(c, units - u), windows) for u in range(0, units, c))
                equal = -(-units // (4 * rounds)) * 4
                if units < 260:
                    assert of(got) == min(of(c) for c in range(equal, min(cap, equal + 63) + 1, 4)), (units, most, windows, got)
    want = {(100, 50, 32): 36, (112, 80, 22): 60, (224, 80, 22): 80, (256, 80, 22): 64, (128, 80, 21): 64, (96, 40, 43): 32, (30, 6, 86): 4}
    assert {k: rules.round_units(*k) for k in want} == want


def test_layers_are_ranked_where_pieces_are_long(rules):
    fn = rules.ranks_by_budget
    fn.restype, fn.argtypes = ctypes.c_bool, [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    for layers, splits, row_bytes in ((28, 2, 256), (64, 64, 256), (2, 9, 128), (28, 18, 512), (64, 1, 256)):
        at = -(-72 * 1024 * layers * splits // row_bytes)                # the sum of the budgets from which they are
        assert not fn(at - 1, layers, splits, row_bytes) and fn(at, layers, splits, row_bytes)
    assert not fn(0, 2, 1, 256) and fn(64 * ((1 << 25) - 1), 64, 64, 512)
    # budgets count, not what a table reaches: eight sequences that keep 300 rows of 128 bf16 columns through any table
    assert not fn(28 * 300, 28, 2, 256) and fn(28 * 1638, 28, 2, 256)


def test_rows_claim_the_cache_where_they_fit_it(rules):
    fn = rules.keeps_rows
    fn.restype, fn.argtypes = ctypes.c_bool, [ctypes.c_longlong, ctypes.c_int]
    for row_bytes in (128, 256, 512):
        assert fn(128_000_000 // row_bytes, row_bytes) and not fn(128_000_000 // row_bytes + 1, row_bytes)
    assert fn(0, 512) and not fn(64 * ((1 << 25) - 1) * 32767, 512)      # (the most that a launch can hand it)
    # 28 layers of 4 heads that keep 1638 rows, whatever a table reaches, and 6554
    assert fn(28 * 4 * 1638, 256) and not fn(28 * 4 * 6554, 256)


def test_grids_begin_at_odd_multiples_of_256_wherever_a_workspace_begins(rules):
    rules.grid_start.restype, rules.grid_start.argtypes = ctypes.c_ulonglong, [ctypes.c_ulonglong]
    rules.grid_slack.restype = ctypes.c_ulonglong
    for base in (0, 256, 512, 4096, (1 << 47) + 256, (1 << 47) + 3840):
        for region in range(0, 2048, 256):
            at = rules.grid_start(base + region)
            assert at % 512 == 256 and 0 <= at - base - region <= rules.grid_slack()


def test_xcds_take_rectangles_that_cover_the_work(rules):
    out = (ctypes.c_int * 4)()
    for first, second in ((1, 1), (3, 180), (5, 1), (7, 9), (11, 23), (48, 30), (86, 28), (158, 15), (16384, 1), (1, 8192)):
        for along in range(4):
            at, most = [], 0
            for xcd in range(8):
                rules.xcd_rectangle(xcd, along, first, second, out)
                f, nf, s, ns = out
                assert nf >= 0 and ns >= 0 and f + nf <= first and s + ns <= second
                most = max(most, nf * ns)
                at.append((f, nf, s, ns))
            assert most == rules.xcd_items(along, first, second)          # (what a launch has workgroups for)
            assert sum(nf * ns for _, nf, _, ns in at) == first * second
            for i, (f, nf, s, ns) in enumerate(at):                       # (no two meet)
                for g, ng, t, nt in at[:i]:
                    assert f + nf <= g or g + ng <= f or s + ns <= t or t + nt <= s or not nf * ns * ng * nt
    # long sequences are cut along the tokens for all XCDs, short ones along the units as well
    assert [rules.xcds_along(*x) for x in ((48, 30, 158, 15), (96, 20, 376, 10), (24, 56, 86, 28), (48, 8, 43, 8))] == [3, 3, 3, 3]
    assert [rules.xcds_along(*x) for x in ((3, 180, 11, 180), (2, 32, 6, 32), (12, 56, 43, 28))] == [0, 1, 2]


def test_waves_have_slots_of_their_own_and_lanes_load_what_their_wave_loads(rules):
    for slots in range(2, 129, 2):
        waves = rules.slot_waves(slots)
        loaded = [[rules.lane_slot(part, lane, slots) for lane in range(16)] for part in range(waves)]
        assert [s for part in range(waves) for s in loaded[part][:slots - 16 * part]] == list(range(slots))
        for part in range(waves):
            # (no wave is empty, and what its lanes past the last slot load is one of its own)
            assert 16 * part < slots and all(16 * part <= s < 16 * part + 16 for s in loaded[part])


def test_rows_of_whole_lines_alone_are_read_past_the_cache(rules):
    keeps = rules.round_keeps_rows
    keeps.restype, keeps.argtypes = ctypes.c_bool, [ctypes.c_longlong, ctypes.c_int]
    for row_bytes in range(16, 1040, 16):
        assert keeps(256_000_000, row_bytes) and keeps(1, row_bytes)
        for much in (256_000_001, 10 ** 10):
            assert keeps(much, row_bytes) == (row_bytes % 128 != 0)


def test_residual_workgroups_take_parts_side_by_side_and_are_resident(rules):
    out = (ctypes.c_int * 7)()

    def plan(wins, tpw, slots, units, dec, bf16):
        rules.residual_plan(wins, tpw, slots, units, *dec, bf16, out)
        return list(out)
    for bf16 in (False, True):
        for slots in (2, 10, 16, 18, 20, 32, 36, 48, 50, 52, 64) + (() if bf16 else (68, 80, 84, 96, 100, 112, 128)):
            parts = rules.slot_waves(slots)
            for tpw in (1, 2, 3, 5, 9, 16):
                for wins in (1, 4, 14, 100, 700):
                    for units in (1, 2, 3, 4, 16, 112, 900):
                        dec = (max(1, wins // 2), -(-units * parts // 4))
                        waves, abreast, blocks, split, once, along, workgroups = plan(wins, tpw, slots, units, dec, bf16)
                        of_unit = (parts if split else 1) * blocks
                        assert 1 <= waves <= 8 and abreast == waves // of_unit and waves == abreast * of_unit
                        assert split == (parts > 1) or (blocks == 1 and (bf16 or (tpw == 1 and units not in (1, 2, 3))))
                        items = rules.xcd_items(along, wins, -(-units // abreast))
                        held = rules.residual_groups(bf16, bool(once), waves, slots)
                        if blocks > 1:
                            held = 32 * (8 // waves)                # (whole workgroups of a compute unit's eight waves)
                        assert workgroups == (items if once else min(items, held)) and workgroups <= held
                        held_once = rules.residual_groups(bf16, True, waves, slots)
                        assert blocks > 1 or once == ((split or parts == 1) and items <= held_once)
    # one layer of a head of 256 fp32 columns and the like: a wave for every part, one turn
    for parts in (5, 6, 8):
        for wins, units in ((14, 1), (43, 4), (21, 4)):
            waves, abreast, _, split, once, _, workgroups = plan(wins, 3, 16 * parts, units, (16, units * parts // 4), False)
            assert (waves, abreast, split, once) == (parts, 1, 1, 1) and workgroups <= 64
    # workgroups of four waves in turn: three of a compute unit where a fifth of a unit's lanes is idle, else two
    for slots, groups in ((4, 96), (12, 96), (14, 64), (16, 64), (20, 96), (24, 96), (28, 64), (32, 64), (52, 64), (64, 64)):
        assert plan(86, 6, slots, 900, (48, 450), False)[4::2] == [0, groups]
        assert rules.residual_groups(False, False, 4, slots) == groups and rules.residual_groups(False, True, 4, slots) == 128
        assert rules.residual_groups(True, False, 4, slots) == rules.residual_groups(True, True, 4, slots) == 64
    assert [rules.residual_groups(False, False, w, s) for w, s in ((3, 36), (3, 48), (5, 68), (6, 84), (7, 100), (8, 120))] == [96, 96, 32, 32, 32, 32]


def test_the_cut_leaves_the_residuals_items_one_turn(rules):
    for dec, res in (((12, 21), (21, 21)), ((12, 21), (22, 21)), ((3, 30), (23, 20)), ((5, 9), (9, 47))):
        for at_once in (16, 32, 64, 128):
            along = rules.xcds_along_at_once(*dec, *res, at_once)
            if rules.xcd_items(3, *res) <= at_once:
                assert rules.xcd_items(along, *res) <= at_once
            else:
                assert along == rules.xcds_along(*dec, *res)
    # 41 units of 4869 tokens: 66 workgroups an XCD by the smaller rectangles alone
    assert [rules.xcd_items(f, 21, 21) for f in (rules.xcds_along(12, 21, 21, 21), rules.xcds_along_at_once(12, 21, 21, 21, 64))] == [66, 63]


def test_decimation_walks_more_tiles_where_the_rows_are_what_it_waits_for(rules):
    rules.decimate_tiles.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool, ctypes.c_int, ctypes.c_longlong]

    def tiles(units, n, m, steps, columns, bf16):
        slots = 2 * columns * (2 if bf16 else 4) // 16
        groups = -(-units * rules.slot_waves(slots) // 4)
        return rules.decimate_tiles(m, groups, steps, bf16, slots, units * 2 * n * columns * (2 if bf16 else 4))
    # large launches, and a chip with few workgroups
    assert tiles(112, 32768, 3072, 10, 128, True) == 4 and tiles(112, 8192, 1536, 6, 128, False) == 4
    assert tiles(1, 512, 96, 6, 64, False) == 1 and tiles(16, 4096, 768, 6, 128, True) == 1
    # weights of four tiles that do not fit the LDS twice
    assert tiles(112, 32768, 2048, 14, 128, True) == 2
    # middle sizes: rows that take longer than a walk ...
    assert tiles(40, 4096, 768, 6, 128, True) == 2 and tiles(48, 4096, 768, 6, 128, True) == 4
    assert tiles(60, 1055, 128, 7, 192, True) == 2 and tiles(90, 700, 128, 4, 128, True) == 2
    assert tiles(132, 1280, 256, 5, 128, True) == 4 and tiles(16, 8192, 1536, 6, 128, True) == 2
    # ... and few bytes: 5 to 20 units of 8 to 32 columns, with 256 to 384 workgroups of the longer walk
    for units, n, m, steps, columns in ((14, 31488, 2048, 13, 16), (15, 30976, 2048, 13, 8), (5, 48896, 4096, 11, 32), (54, 7348, 512, 13, 16),
                                        (111, 3901, 256, 13, 24), (13, 13729, 2048, 7, 8)):
        assert tiles(units, n, m, steps, columns, True) == 1


def test_selections_copy_rows_where_a_workgroups_share_is_short(rules):
    rules.copy_groups.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong, ctypes.c_int, ctypes.c_bool]

    def groups(B, L, H, n, d, rho, element, shared, paged):
        return rules.copy_groups(B * L if shared else B * L * H, L, n, H if shared else 1, B * H * int(rho * L * n), d * element // 16, paged)
    # one launch: a layer of a short prompt, four layers of 4096 tokens, sixteen sets of 1280, few heads alike
    assert groups(1, 1, 2, 512, 64, 0.2, 4, False, False) == 32 and groups(1, 4, 4, 4096, 128, 0.2, 2, False, False) == 256
    assert groups(1, 4, 4, 1280, 128, 0.2, 2, False, True) == 256 and groups(1, 6, 2, 2048, 64, 0.1, 2, True, True) == 96
    # two: many sets, long sequences, long shares
    assert groups(1, 28, 4, 8192, 128, 0.2, 2, False, False) == groups(1, 1, 4, 32768, 128, 0.2, 2, False, False) == 0
    assert groups(1, 2, 4, 16384, 128, 0.2, 2, False, False) == 0
    # ... shares of more than two and a half turns of a workgroup's threads through tables, or four
    for case in ((1, 9, 4, 567, 256, 0.328, 2, True), (3, 5, 8, 748, 128, 0.243, 2, True), (3, 2, 2, 577, 256, 0.311, 4, True),
                 (1, 6, 2, 849, 256, 0.328, 4, False), (1, 2, 8, 2162, 128, 0.043, 4, True)):
        assert groups(*case, True) == 0, case
    assert groups(1, 12, 4, 945, 128, 0.397, 2, False, False) == 0
    # ... and sets whose heads' scores each of their workgroups would read
    for case in ((2, 18, 8, 8907, 8, 0.027, 4, True, False), (1, 24, 4, 13488, 8, 0.292, 2, True, False), (2, 28, 4, 13639, 8, 0.026, 2, True, True)):
        assert groups(*case) == 0, case


def test_places_of_a_butterfly_are_sums_where_the_transforms_say_so(rules):
    rules.pads_apart.restype = ctypes.c_bool
    for group in (2, 4, 8, 16, 32):
        def place(i):
            return i + i // group
        for radix in (2, 3, 4, 6, 8, 12, 16, 24, 32, 48):
            for done in (1, 8, 16, 32, 64):
                firsts = [t // done * done * radix + t % done for t in range(4 * max(group, done))]
                holds = all(place(f + q * done) == place(f) + place(q * done) for f in firsts for q in range(radix))
                assert holds or not rules.pads_apart(radix, done, group), (radix, done, group)
                if done == 1:
                    assert holds == rules.pads_apart(radix, done, group), (radix, group)
    assert not rules.pads_apart(6, 1, 8) and not rules.pads_apart(12, 1, 16) and rules.pads_apart(16, 1, 16) and rules.pads_apart(32, 1, 16)
