"""The device code that divides the verify attention's work, run on the host under
AddressSanitizer and UndefinedBehaviorSanitizer (CPU only).

csrc/attn_plan.h and the headers it needs are built with g++ against a stand-in for
hip_runtime.h (tests/sanitize/host_hip) and driven by tests/sanitize/attn_plan_driver.cpp."""
import os
import subprocess

import pytest

import attn_words
from test_sanitizers import ENV_SAN, ROOT, SAN, _have, _run

pytestmark = pytest.mark.skipif(not _have("g++"), reason="g++ not found")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = tmp_path_factory.mktemp("attn_plan") / "attn_plan_driver"
    san = os.path.join(ROOT, "tests", "sanitize")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", *SAN, "-pthread",
                    "-I", os.path.join(san, "host_hip"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2607_25852_amd", "csrc"),
                    os.path.join(san, "attn_plan_driver.cpp"), "-o", str(exe)], check=True)
    return str(exe)


def test_plan_code_on_the_host(driver):
    r = _run([driver])
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-4000:]
    assert r.stdout.startswith("ok"), r.stdout


@pytest.mark.parametrize("shape", attn_words.SHAPES)
def test_run_on_words_stays_in_bounds(driver, shape):
    """The words that the GPU test of runs without a plan puts into the workspace: every piece they
    make lies in the batch, its request and the partial results."""
    Hq, Hkv, d, page, b, ctx = shape
    _, qo, kv = attn_words.case(shape)
    R, G, top = len(ctx), Hq // Hkv, int(kv.max())
    ranges = attn_words.ranges_of(Hq, Hkv, b, R, top)
    blocks = -(-G * b // (256 if G * b > 128 else 128))
    pieces = {}
    for kind in attn_words.KINDS:
        count, rec = attn_words.words(kind, ranges, R, b, qo, kv)
        nums = [R, b, int(qo[-1]), top, G, blocks, Hkv, ranges, *qo, *kv, count, *rec.ravel()]
        r = subprocess.run([driver, "words"], input=" ".join(str(int(v)) for v in nums), capture_output=True, text=True,
                           env=dict(os.environ, **ENV_SAN), timeout=120)
        assert r.returncode == 0, (kind, r.stdout[-500:] + r.stderr[-2000:])
        pieces[kind] = int(r.stdout.split()[1])
    assert pieces["bytes ff"] == pieces["negative count"] == 0, pieces
    assert R == 1 or (pieces["stray tiles"] > 0 and sum(pieces[k] for k in pieces if k.startswith("mix")) > 0), pieces


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
