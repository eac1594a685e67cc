"""bench.py's profile summaries know the kernels that run (CPU only).

The names are taken from the sources: a kernel that is renamed or added without its summary fails
here. The digest beside a recorded traffic figure changes with every source that decides it."""
import csv
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

KERNEL = re.compile(r"__global__\s+__launch_bounds__\([^)]*\)\s*void\s+(\w+)\s*\(")


def kernels_of(source):
    return KERNEL.findall(open(os.path.join(bench.CSRC, source)).read())


def test_every_attention_kernel_is_known():
    bf16 = set(kernels_of("attn.hip") + kernels_of("attn_list.hip")) - {"attn_f32_kernel"}
    assert bf16 == set(bench.ATTN_KERNELS)
    accept = set(kernels_of("accept.hip"))
    assert set(bench.ACCEPT_KERNELS) <= accept


def test_no_name_is_part_of_another():
    """The summaries look names up as parts of the profiler's full names."""
    names = bench.ATTN_KERNELS + bench.ACCEPT_KERNELS
    assert not [(a, b) for a in names for b in names if a != b and a in b]


@pytest.mark.parametrize("division", ["ranges", "list"])
def test_trace_and_traffic_find_the_attention(tmp_path, division):
    plan, run, merge = bench.ATTN_DIVISIONS[division]
    full = {k: f"void sv::(anonymous namespace)::{k}<128>(sv::AttnArgs)" for k in (plan, run, merge)}
    stats = tmp_path / "run_kernel_stats.csv"
    with open(stats, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Name", "Calls", "AverageNs", "MinNs", "MaxNs", "Percentage"])
        for k, ns in ((plan, 4000), (run, 200000), (merge, 6000)):
            w.writerow([full[k], 10, ns, ns, ns, 1.0])
    text = bench.summarize_trace(str(stats))
    assert "206.0 us" in text and "4.0 us" in text and division in text
    neg = "void at::native::neg_kernel_cuda<float>"
    for d, counter, copy in (("fetch", "FETCH_SIZE", bench.COPY_BYTES / 2048), ("write", "WRITE_SIZE", bench.COPY_BYTES / 1024)):
        os.makedirs(tmp_path / d)
        with open(tmp_path / d / "run_counter_collection.csv", "w", newline="") as f:
            w = csv.writer(f)
            w.writerow(["Kernel_Name", "Counter_Name", "Counter_Value"])
            w.writerow([neg, counter, copy])
            for k, kib in ((run, 1000), (run, 1000), (merge, 24), (merge, 24)):
                w.writerow([full[k], counter, kib])
    text = bench.summarize_traffic(str(tmp_path / "fetch"), str(tmp_path / "write"))
    assert "- calls: 2" in text
    assert f"- traffic_bytes_per_call: {1024 * 1024 * 3}" in text  # fetch counts twice, write once


def test_digest_covers_every_attention_source(tmp_path, monkeypatch):
    includes = {m for f in ("attn.hip", "attn_list.hip") for m in
                re.findall(r'#include "([^"]+)"', open(os.path.join(bench.CSRC, f)).read())}
    headers = {h for h in includes if h.startswith("attn")} | {"rows.h"}
    assert {"attn.hip", "attn_list.hip", "sv_host.cpp"} | headers <= set(bench.ATTN_SOURCES)
    for name in bench.ATTN_SOURCES:
        (tmp_path / name).write_bytes(open(os.path.join(bench.CSRC, name), "rb").read())
    monkeypatch.setattr(bench, "CSRC", str(tmp_path))
    before = bench.attn_source_digest()
    for name in bench.ATTN_SOURCES:
        old = (tmp_path / name).read_bytes()
        (tmp_path / name).write_bytes(old + b"\n")
        assert bench.attn_source_digest() != before, name
        (tmp_path / name).write_bytes(old)
    assert bench.attn_source_digest() == before
