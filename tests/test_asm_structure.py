"""Structure of the compiled work loops (gfx950 assembly built on the CPU, no GPU).

A persistent kernel claims its next work item with `if (tid == 0) item = atomicAdd(...)`
followed by a workgroup barrier. If the compiler threads that lane-divergent test through a
loop back edge, the barrier ends up in an inner loop that lane 0 of wave 0 has left; the
hardware barrier counts waves, so the other lanes pass it without the claim and the loop
never ends. This test fails if the first barrier after any claim lies in a different loop
than the claim itself."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_25852_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

LABEL = re.compile(r"^(\.LBB\d+_\d+):|^; %bb\.(\d+):")
HEADER = re.compile(r"=>\s*This (?:Inner )?Loop Header: Depth=(\d+)")
IN_LOOP = re.compile(r"in Loop: Header=(BB\d+_\d+) Depth=(\d+)")


def _assemble(src, tmp_path):
    out = tmp_path / (os.path.splitext(src)[0] + ".s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", os.path.join(CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text().split("\n")


def _functions(lines):
    """(name, body lines) of every kernel in an assembly listing."""
    out, name, body = [], None, []
    for l in lines:
        m = re.match(r"^(_Z\S+):", l)
        if m:
            name, body = m.group(1), []
            continue
        if name and l.startswith(".Lfunc_end"):
            out.append((name, body))
            name = None
            continue
        if name:
            body.append(l)
    return out


def _loop_of_each_line(body):
    """innermost loop header of the block holding each line (None outside loops); a block's
    loop annotation is on its label line or on the comment lines right after it"""
    res, cur_loop = [], None
    for n, l in enumerate(body):
        m = LABEL.match(l)
        if m:
            blk = m.group(1)[2:] if m.group(1) else None  # ".LBB2_5" -> "BB2_5"
            notes = [l]
            k = n + 1
            while k < len(body) and body[k].lstrip().startswith(";"):
                notes.append(body[k])
                k += 1
            note = " ".join(notes)
            h = HEADER.search(note)
            il = IN_LOOP.search(note)
            if h and blk:
                cur_loop = blk
            elif il:
                cur_loop = il.group(1)
            else:
                cur_loop = None
        res.append(cur_loop)
    return res


def claims_and_barriers(lines, kernel_pattern):
    """[(kernel, loop of the claim, loop of the next barrier)] for every global atomic add
    that is followed by a barrier"""
    found = []
    for name, body in _functions(lines):
        if not re.search(kernel_pattern, name):
            continue
        loops = _loop_of_each_line(body)
        for i, l in enumerate(body):
            if "global_atomic_add" not in l:
                continue
            j = next((k for k in range(i + 1, len(body)) if "s_barrier" in body[k]), None)
            if j is not None:
                found.append((name, loops[i], loops[j]))
    return found


def test_attention_claim_and_barrier_share_a_loop(tmp_path):
    lines = _assemble("attn.hip", tmp_path)
    found = claims_and_barriers(lines, r"attn_bf16_kernel")
    assert len(found) >= 4, found  # one claim per instantiated persistent kernel
    for name, claim_loop, barrier_loop in found:
        assert claim_loop is not None and claim_loop == barrier_loop, (name, claim_loop, barrier_loop)


def test_list_claim_and_barrier_share_a_loop(tmp_path):
    """The same for the work list's kernels, which always claim: four shapes of tile and page,
    each with and without whole-tile waves."""
    found = claims_and_barriers(_assemble("attn_list.hip", tmp_path), r"attn_list_kernel")
    assert len({name for name, _, _ in found}) == 8, found
    for name, claim_loop, barrier_loop in found:
        assert claim_loop is not None and claim_loop == barrier_loop, (name, claim_loop, barrier_loop)


def test_no_other_file_claims_work(tmp_path):
    """The two tests above name every source whose kernels loop over claimed items."""
    loops = [f for f in sorted(os.listdir(CSRC)) if f.endswith(".hip") and "atomicAdd(&ctr[" in open(os.path.join(CSRC, f)).read()]
    assert loops == ["attn.hip", "attn_list.hip"], loops


def test_checker_flags_a_threaded_claim():
    """The checker on a hand-written listing with the miscompiled shape: the claim in the
    outer loop, its barrier in an inner loop entered from the unit's latch."""
    listing = """_ZN2sv6kernelEv:
.LBB2_129:                              ;   in Loop: Header=BB2_130 Depth=1
\ts_cbranch_execz .LBB2_485
.LBB2_130:                              ; =>This Loop Header: Depth=1
\ts_and_saveexec_b64 s[0:1], s[42:43]
; %bb.132:                              ;   in Loop: Header=BB2_130 Depth=1
\tglobal_atomic_add v3, v73, v3, s[94:95] sc0
.LBB2_134:                              ;   in Loop: Header=BB2_130 Depth=1
\ts_branch .LBB2_137
.LBB2_137:                              ;   Parent Loop BB2_130 Depth=1
                                        ; =>  This Loop Header: Depth=2
\ts_barrier
.Lfunc_end0:
"""
    lines = listing.split("\n")
    found = claims_and_barriers(lines, r"kernel")
    assert found == [("_ZN2sv6kernelEv", "BB2_130", "BB2_137")]


def test_vector_loads_keep_their_alignment(tmp_path):
    """Rows of odd vocabularies start at any element: the acceptance's 16-byte loads are made
    through types of the element's alignment. A pointer to one passed on as a 16-byte aligned
    vector is an error in the build, and the loads are single 16-byte instructions all the same."""
    from paper_2607_25852_amd import build
    assert "-Werror=align-mismatch" in build.COMMON
    src = tmp_path / "planted.hip"
    src.write_text("typedef float v4 __attribute__((ext_vector_type(4)));\n"
                   "typedef v4 u4 __attribute__((aligned(4)));\n"
                   "template <typename V> __device__ V get(const V* p) { return __builtin_nontemporal_load(p); }\n"
                   "__global__ void k(const float* p, float* q) { q[0] = get((const u4*)(p + 1))[0]; }\n")
    r = subprocess.run([HIPCC, "-x", "hip", *build.COMMON, "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert r.returncode != 0 and "align-mismatch" in r.stderr, r.stderr[-2000:]
    r = subprocess.run([HIPCC, "-x", "hip", *build.COMMON, "-fsyntax-only", os.path.join(CSRC, "accept.hip")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    for name, body in _functions(_assemble("accept.hip", tmp_path)):
        if re.search(r"rowstats_kernel|argmax_kernel|dstats_chunk_kernel", name):
            assert sum("global_load_dwordx4" in l and " nt" in l for l in body) >= 8, name


def test_chunk_loads_are_in_flight_together(tmp_path):
    """The statistics passes issue a chunk's four 16-byte loads back to back: no wait between them,
    which would make two round trips to memory of one."""
    seen = 0
    for name, body in _functions(_assemble("accept.hip", tmp_path)):
        if not re.search(r"rowstats_kernel|dstats_chunk_kernel", name):
            continue
        seen += 1
        at = [i for i, l in enumerate(body) if "global_load_dwordx4" in l and " nt" in l]
        assert len(at) % 4 == 0, (name, len(at))
        for g in range(0, len(at), 4):
            between = body[at[g]:at[g + 3]]
            assert not any("s_waitcnt" in l and "vmcnt" in l for l in between), (name, between)
    assert seen == 4, seen
