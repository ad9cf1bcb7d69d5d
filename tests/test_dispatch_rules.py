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
int round_units(int units, int most) { return fc::round_units(units, most); }
unsigned long long grid_start(unsigned long long at) { return fc::grid_start(at); }
unsigned long long grid_slack() { return fc::kGridSlack; }
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


def test_rounds_are_as_few_and_as_equal_as_whole_sets_allow(rules):
    for most in list(range(1, 200)) + [480, 1000]:
        for units in list(range(1, 400)) + [896, 4000, 32767]:
            got = rules.round_units(units, most)
            if units <= most or most < 4:
                assert got == min(units, most)
                continue
            cap = most // 4 * 4
            rounds = -(-units // cap)
            assert 4 <= got <= cap and got % 4 == 0, (units, most, got)
            assert -(-units // got) == rounds, (units, most, got)       # (no round for what is left over)
            assert (got - 4) * rounds < units, (units, most, got)       # (a set less in each would not do)
    assert [rules.round_units(*x) for x in ((100, 50), (112, 80), (132, 66), (26, 15), (30, 6))] == [36, 56, 44, 12, 4]


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
