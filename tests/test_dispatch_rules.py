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
