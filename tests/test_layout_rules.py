"""The layouts and tile lists of the library's host code, on the CPU, in a host-only
build with AddressSanitizer and UndefinedBehaviorSanitizer: rules and invariants in
tests/sanitize/layout_driver.cpp."""
from __future__ import annotations

import os
import subprocess

import pytest

from paper_2512_01032_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = os.path.join(ROOT, "tests", "sanitize")


def test_layout_rules(tmp_path):
    hc = build.hipcc()
    if not os.path.exists(os.path.join(SAN, "layout_driver.cpp")):
        pytest.skip("driver not in this copy of the tree")
    san = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-omit-frame-pointer"]
    objs = []
    for src in (os.path.join(build.CSRC, "lattice_host.hip"), os.path.join(SAN, "layout_driver.cpp"),
                os.path.join(SAN, "launch_stubs.cpp")):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.check_call([hc, "-x", "hip", "--cuda-host-only", "-O1", "-g", "-std=c++17", "-fPIC", "-w"] +
                              san + ["-c", src, "-o", obj])
        objs.append(obj)
    exe = str(tmp_path / "layout_driver")
    subprocess.check_call([hc, "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                           "-o", exe] + objs)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    env.pop("LBM_TILE_Z", None)
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    print(r.stdout[-4000:], r.stderr[-3000:])
    assert r.returncode == 0 and r.stdout.strip().endswith("OK")
    assert "ERROR: AddressSanitizer" not in r.stderr and "runtime error" not in r.stderr
