"""States of the matching solver lie one after the other in LDS, each beginning
with 64-bit arrays: the size of one keeps the next aligned, at the capacity of
every code and of every launch."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include "include/mcmcdec.h"
#define MW_FN inline
#define MW_HD inline
#include "paper_1302_2669_amd/csrc/mwpm_solver.h"
int main() {
  for (int cap = 4; cap <= mcmc::mw::capacity(MCMC_L_MAX); cap += 4)
    printf("%d %zu\\n", cap, mcmc::mw::region_bytes(cap));
}
"""


def test_regions_keep_the_next_state_aligned(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    src, exe = tmp_path / "regions.cpp", tmp_path / "regions"
    src.write_text(SOURCE)
    subprocess.run([gxx, "-std=c++17", "-I", ROOT, "-o", str(exe), str(src)], check=True,
                   capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    sizes = {int(a): int(b) for a, b in (line.split() for line in out.splitlines())}
    assert {8, 64, 88, 156, 604} <= set(sizes)
    assert all(size % 8 == 0 and size >= 83 * cap for cap, size in sizes.items())
