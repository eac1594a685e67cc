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


@pytest.mark.parametrize("R,total_q,b,Hq,Hkv,d,max_kv,split", [
    (4, 16, 16, 64, 8, 128, 65536, 2048), (1, 16, 16, 8, 8, 64, 4096, 64), (20, 100, 8, 32, 4, 128, 131072, 8192),
    (64, 512, 16, 64, 8, 128, 32768, 4096), (3, 12, 4, 16, 2, 64, 1000, 1024)])
def test_workspace_of_a_given_split(R, total_q, b, Hq, Hkv, d, max_kv, split):
    """A given split takes one partial result per split and packed row, and the list of items."""
    from paper_2607_25852_amd import binding as B
    desc = B.attn_desc(R, total_q, b, Hq, Hkv, d, 64, -(-max_kv // 64), 1 << 16, max_kv, B.SV_BF16, kv_split=split)
    splits = -(-max_kv // split)
    partials = splits * total_q * Hq * (d + 1) * 4 if splits > 1 else 0
    items = R * splits * 4
    assert B.attn_workspace_size(desc) <= partials + items + 2 * 256 + 12
