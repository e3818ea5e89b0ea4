"""Which contexts' resident launches may run on the device together (csrc/resident_admission.hpp),
compiled for the host alone: launches that may be running at the same time must all fit, also where a
context has gone over to a smaller plan while its larger launches are still queued."""
import shutil
import subprocess

import pytest

from paper_2005_09323_amd import build as libbuild

PROGRAM = r"""
#include "resident_admission.hpp"
#include <cstdio>
using namespace lbm;
static int failed = 0;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); failed = 1; } } while (0)
int main() {
    const ResidentUse big{256, 1}, small{8, 1}, half{128, 1}, pairs{300, 2}, mixed = either_of(half, pairs);
    // one context alone: always
    CHECK(side_by_side({big}, 256) && side_by_side({mixed}, 256) && side_by_side({}, 256));
    // as many workgroups as the device has places, not one more
    CHECK(side_by_side({half, half}, 256) && !side_by_side({half, half, small}, 256));
    CHECK(side_by_side({pairs, ResidentUse{212, 2}}, 256) && !side_by_side({pairs, ResidentUse{213, 2}}, 256));
    // workgroups of different sizes share no count of places
    CHECK(!side_by_side({small, ResidentUse{8, 2}}, 256) && !side_by_side({mixed, small}, 256) && !side_by_side({small, mixed}, 256));
    // a context whose large launches may still be running steps fewer members now
    const ResidentUse both = either_of(big, small);
    CHECK(both.blocks == 256 && both.places == 1 && !side_by_side({half, both}, 256));
    CHECK(either_of(pairs, small).places == 0 && mixed.places == 0 && mixed.blocks == 300);
    return failed;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_launches_that_may_run_together_fit(tmp_path):
    src, exe = tmp_path / "admission.cpp", tmp_path / "admission"
    src.write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", libbuild.CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

