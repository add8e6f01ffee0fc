"""The guard on the chain launches' queue counters: the headers compile, and no
longer do with one counter less than a plan's launches use."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("slots,compiles", [(16, True), (15, False)])
def test_a_counter_too_few_does_not_compile(tmp_path, slots, compiles):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    csrc = tmp_path / "paper_1302_2669_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_1302_2669_amd", "csrc"), csrc)
    header = csrc / "host_common.h"
    text = header.read_text()
    assert text.count("kQueueSlots = 16;") == 1
    header.write_text(text.replace("kQueueSlots = 16;", f"kQueueSlots = {slots};"))
    (csrc / "one.cpp").write_text('#include "host_common.h"\n')
    res = subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-fsyntax-only",
                          str(csrc / "one.cpp")], capture_output=True, text=True, timeout=120)
    assert (res.returncode == 0) == compiles, res.stderr
    if not compiles:
        assert "static assertion failed" in res.stderr or "static_assert failed" in res.stderr
