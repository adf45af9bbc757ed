"""The library's sizing rules (plan.cpp) on the CPU: tests/host/plan_check.cpp
built with g++, one check per test."""

from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("plan") / "plan_check")
    host = os.path.join(ROOT, "tests", "host")
    cmd = [gxx, "-std=c++17", "-O1", "-I", os.path.join(host, "include"),
           os.path.join(host, "plan_check.cpp"),
           os.path.join(ROOT, "paper_2606_18600_amd", "csrc", "plan.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


@pytest.mark.parametrize("check", ["prefill_parts", "stream", "half_round", "row_tail", "gate_up",
                                   "swiglu_tail", "rows192", "decode_splits"])
def test_sizing_rules(exe, check):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stderr[-2000:]
