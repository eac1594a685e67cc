"""The device code that divides the verify attention's work, run on the host under
AddressSanitizer and UndefinedBehaviorSanitizer (CPU only).

csrc/attn_plan.h and the headers it needs are built with g++ against a stand-in for
hip_runtime.h (tests/sanitize/host_hip) and driven by tests/sanitize/attn_plan_driver.cpp."""
import os
import subprocess

import pytest

from test_sanitizers import ROOT, SAN, _have, _run

pytestmark = pytest.mark.skipif(not _have("g++"), reason="g++ not found")


def test_plan_code_on_the_host(tmp_path):
    exe = tmp_path / "attn_plan_driver"
    san = os.path.join(ROOT, "tests", "sanitize")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", *SAN, "-pthread",
                    "-I", os.path.join(san, "host_hip"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2607_25852_amd", "csrc"),
                    os.path.join(san, "attn_plan_driver.cpp"), "-o", str(exe)], check=True)
    r = _run([str(exe)])
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-4000:]
    assert r.stdout.startswith("ok"), r.stdout
