"""sv_verify_attn_run over ranges on a workspace that holds no plan: arbitrary words in the place of
the plan (attn_words.py; the CPU test runs the same words through the plan's own code) and the plan
of other key counts. The results are unspecified, but the call succeeds, every write stays inside
the outputs and the workspace, and a plan built afterwards gives sv_verify_attn's results bit for
bit."""
import dataclasses

import numpy as np
import pytest

import attn_words
from gpu_util import say
from test_gpu_attn import dev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

PAD = 4096  # guard elements on either side


def guarded(torch, n, dtype, value):
    buf = torch.full((n + 2 * PAD,), value, dtype=dtype, device="cuda")
    return buf, buf[PAD:PAD + n]


@pytest.mark.parametrize("shape", attn_words.SHAPES)
def test_run_without_its_plan_over_ranges(dev, shape):  # noqa: F811
    torch = dev
    from paper_2607_25852_amd import binding as B, synth
    from paper_2607_25852_amd.round import to_dev
    Hq, Hkv, d, page, b, ctx = shape
    R = len(ctx)
    k, qo, kvl = attn_words.case(shape)
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"words_h{Hq}_{Hkv}_d{d}_p{page}", R=R, b=b, dtype="bf16",
                              Hq=Hq, Hkv=Hkv, d=d, page=page, kv=("list",) + tuple(ctx))
    L = synth.kv_context_lengths(cfg)
    kv = synth.make_kv(cfg, L)
    rows = int(qo[-1])
    desc = B.attn_desc(R, rows, b, Hq, Hkv, d, page, kv["page_table"].shape[1], kv["num_pages"], int(kvl.max()), B.SV_BF16)
    ranges = attn_words.ranges_of(Hq, Hkv, b, R, int(kvl.max()))
    size = B.attn_workspace_size(desc)
    off_ctr = size - 12
    off_cuts = off_ctr - -(-(ranges + 1) * 32 // 256) * 256
    assert off_ctr % 256 == 0 and off_cuts > 0
    ws_buf, ws = guarded(torch, size, torch.uint8, 0x5A)
    out_buf, out = guarded(torch, rows * Hq * d, torch.bfloat16, -3.0)
    lse_buf, lse = guarded(torch, rows * Hq, torch.float32, -3.0)
    q, kc, vc, pt, d_qo, d_kv = (to_dev(x) for x in (synth.pack_rows(kv["q_full"], qo), kv["k_cache"], kv["v_cache"],
                                                     kv["page_table"], qo, kvl))

    def run(key_counts=d_kv):
        B.verify_attn_run(desc, q, kc, vc, pt, d_qo, key_counts, out.view(rows, Hq, d), lse.view(rows, Hq), ws)
        torch.cuda.synchronize()

    def guards():
        for buf, v in ((ws_buf, 0x5A), (out_buf, -3.0), (lse_buf, -3.0)):
            assert bool((buf[:PAD] == v).all()) and bool((buf[-PAD:] == v).all())

    B.verify_attn(desc, q, kc, vc, pt, d_qo, d_kv, out.view(rows, Hq, d), lse.view(rows, Hq), ws)
    torch.cuda.synchronize()
    ctr = ws[off_ctr:].view(torch.int32).cpu().tolist()
    assert 1 <= ctr[0] <= ranges and ctr[1:] == [0, 0]  # (the place of the plan)
    ref_out, ref_lse = out.clone(), lse.clone()
    for kind in attn_words.KINDS:
        count, rec = attn_words.words(kind, ranges, R, b, qo, kvl)
        ws[off_cuts:off_cuts + rec.nbytes].copy_(torch.from_numpy(rec.view(np.uint8).ravel()))
        ws[off_ctr:].copy_(torch.from_numpy(np.array([count, 0, 0], np.int32).view(np.uint8)))
        say("attention on words", cfg.name, kind)
        run()
        guards()
    # the plan of other key counts
    other = to_dev((k + (kvl - k) // 2).astype(np.int32))
    B.verify_attn_plan(desc, d_qo, other, ws)
    say("attention on another plan", cfg.name)
    run()
    guards()
    B.verify_attn_plan(desc, d_qo, d_kv, ws)
    out.fill_(-5.0)
    for _ in range(2):
        run()
        assert torch.equal(out, ref_out) and torch.equal(lse, ref_lse)
    guards()
