"""A given kv_split cuts each request's own context: a request's results are the same bits alone
and in any batch, below and above the number of units that takes the work list by itself. Without
one, the same call twice gives the same bits."""
import dataclasses

import numpy as np
import pytest

from gpu_util import say
from test_gpu_attn import dev, run_gpu_attn  # noqa: F401  (dev: fixture)

pytestmark = pytest.mark.gpu

# (Hq, Hkv, d, page, b, contexts, kv_split): the first request is compared
CASES = [
    (16, 4, 128, 64, 8, (1000, 700, 64, 3), 256),
    (16, 2, 64, 16, 16, (900, 2000, 5), 128),
    (32, 2, 128, 64, 16, (777, 1500), 192),           # whole-tile waves
    (8, 4, 64, 4, 4, (450, 33, 700), 64),             # a page per lane
    (8, 8, 128, 64, 4, (500,) + (70,) * 63, 192),     # 512 units
]


@pytest.mark.parametrize("Hq,Hkv,d,page,b,ctx,split", CASES)
def test_given_split_is_the_requests_own(dev, Hq, Hkv, d, page, b, ctx, split):  # noqa: F811
    from paper_2607_25852_amd import binding as B, synth
    from paper_2607_25852_amd.round import to_dev
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"split_h{Hq}_{Hkv}_d{d}_p{page}_s{split}", R=len(ctx), b=b,
                              dtype="bf16", Hq=Hq, Hkv=Hkv, d=d, page=page, kv=("list",) + tuple(ctx))
    L = synth.kv_context_lengths(cfg)
    kv = synth.make_kv(cfg, L, fill_unused=np.nan, q_scale=4.0)
    depths = np.array([b - i % b for i in range(len(ctx))])
    qo = synth.indptr_from_depths(depths)
    say("attn split", cfg.name)
    _, kvl, o, l = run_gpu_attn(dev, cfg, kv, qo, L, kv_split=split)
    # the first request alone, in the same cache: same max_kv_len and page-table width
    page_table = np.ascontiguousarray(kv["page_table"][:1])
    k0 = int(depths[0])
    desc = B.attn_desc(1, k0, b, Hq, Hkv, d, page, page_table.shape[1], kv["num_pages"], int(kvl.max()),
                       B.SV_BF16, kv_split=split)
    torch = dev
    out = torch.full((k0, Hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((k0, Hq), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(max(B.attn_workspace_size(desc), 256), dtype=torch.uint8, device="cuda")
    B.verify_attn(desc, to_dev(synth.pack_rows(kv["q_full"][:1], qo[:2])), to_dev(kv["k_cache"]), to_dev(kv["v_cache"]),
                  to_dev(page_table), to_dev(np.ascontiguousarray(qo[:2], np.int32)),
                  to_dev(kvl[:1].astype(np.int32)), out, lse, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.float().cpu().numpy(), o[:k0].astype(np.float32))
    np.testing.assert_array_equal(lse.cpu().numpy(), l[:k0].astype(np.float32))


@pytest.mark.parametrize("Hq,Hkv,d,page,b,ctx,split", CASES[:4])
def test_own_division_repeats(dev, Hq, Hkv, d, page, b, ctx, split):  # noqa: F811
    from paper_2607_25852_amd import synth
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"again_h{Hq}_{Hkv}_d{d}_p{page}", R=len(ctx), b=b,
                              dtype="bf16", Hq=Hq, Hkv=Hkv, d=d, page=page, kv=("list",) + tuple(ctx))
    L = synth.kv_context_lengths(cfg)
    kv = synth.make_kv(cfg, L)
    qo = synth.indptr_from_depths(np.array([b - i % b for i in range(len(ctx))]))
    say("attn repeat", cfg.name)
    first, second = (run_gpu_attn(dev, cfg, kv, qo, L) for _ in range(2))
    np.testing.assert_array_equal(first[2], second[2])
    np.testing.assert_array_equal(first[3], second[3])
