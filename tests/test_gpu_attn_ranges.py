"""The plans of the bf16 attention at their edges, every (row, head) against the fp64 oracle.

Ranges of equal cost: head counts that do not divide the compute units, pages that hold a whole
tile, a DMA segment of one or less, contexts of more pages than are staged at once, cuts at and
next to the ends of units, more items than workgroups, and several row blocks. The work list:
the first sizes that take it, next to the last ones that do not. Gates of test_gpu_attn.py.
"""
import dataclasses

import numpy as np
import pytest

from gpu_util import say
from test_gpu_attn import check, dev, run_gpu_attn  # noqa: F401  (dev: fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, d, page, b, contexts, kv_split)
    (6, 3, 128, 64, 4, (700, 63, 64, 65), 0),          # 85 ranges of 3 heads: the last wave partly empty
    (14, 7, 64, 32, 8, (1500, 1, 129), 0),
    (48, 24, 128, 64, 2, (900, 300), 0),               # 10 ranges of 24 heads
    (4, 2, 128, 8, 4, (8300, 20), 0),                  # a page per segment, 1038 pages
    (4, 2, 64, 8, 4, (8300, 20), 0),
    (4, 2, 64, 4, 4, (4200, 7), 0),                    # a page per lane, 1050 pages
    (4, 2, 128, 1, 4, (1100, 1024), 0),
    (5, 5, 128, 2, 4, (2500, 3), 0),
    (8, 1, 128, 64, 16, (64 * 6, 64 * 6, 64 * 7), 0),  # units of just the shortest range
    (8, 8, 128, 64, 16, (64 * 13 - 16,) * 4, 0),       # 65 to 128 rows per kv-head, equal lengths
    (40, 1, 64, 64, 16, (500, 900), 0),                # whole-tile waves, three row blocks
    (4, 4, 128, 64, 4, (6000, 100, 64), 64),           # a given split: more items than workgroups
    (100, 100, 64, 64, 4, (2300,), 0),                 # 11 ranges of 100 heads: more items than workgroups, claims
    (56, 56, 128, 16, 2, (3000, 700), 0),              # 19 ranges of 56 heads, 112 units
    (57, 57, 128, 16, 2, (3000, 700), 0),              # 114 units of an uneven head count: the list
    (44, 44, 64, 64, 2, (4090,), 0),                   # 64 tiles: ranges
    (44, 44, 64, 64, 2, (4100,), 0),                   # 65 tiles: the list, three splits
    (32, 4, 128, 64, 16, (64 * 8 - 16,) + (60,) * 15, 0),   # 64 units of at most 8 tiles: the list, one split each
    (32, 4, 128, 64, 16, (64 * 8 - 15,) + (60,) * 15, 0),   # 9 tiles: ranges, a short line
    (32, 4, 128, 64, 16, (64 * 2 - 16, 40, 20, 7), 0),      # 16 units: ranges
    (16, 4, 128, 64, 4, (64 * 30, 40, 200, 333), 0),        # a short line with one long unit
    (64, 8, 128, 64, 16, (64 * 9, 7, 500, 90), 0),          # 32 units, 65 to 128 rows, 10 tiles: ranges
    (32, 8, 64, 16, 8, (64 * 16 - 8,) + (300,) * 15, 0),    # 128 units of at most 16 tiles: the list
    (32, 8, 64, 16, 8, (64 * 16 - 7,) + (300,) * 15, 0),    # 17 tiles: ranges
    (32, 8, 64, 16, 8, (64 * 10 - 8,) + (300,) * 15, 0),    # up to 64 rows, 10 tiles: ranges
    (32, 8, 64, 16, 8, (64 * 10 - 7,) + (300,) * 15, 0),    # 11 tiles: the list
    (32, 2, 128, 64, 16, (64 * 8 - 16,) + (50,) * 31, 0),   # 64 units of whole-tile waves: the list
    (16, 8, 128, 64, 4, (64 * 4 - 4,) + (60,) * 32, 0),     # 264 units of at most 4 tiles: ranges
    (16, 8, 128, 64, 4, (64 * 4 - 3,) + (60,) * 32, 0),     # 5 tiles: the list
    (4, 4, 64, 1, 4, (1100,) + (50,) * 39, 0),              # 160 units, two splits on pages of one token: ranges
    (8, 8, 128, 64, 3, tuple(range(40, 40 + 63)), 0),  # 504 units: ranges
    (8, 8, 128, 64, 3, tuple(range(40, 40 + 64)), 0),  # 512 units: the list
]


@pytest.mark.parametrize("Hq,Hkv,d,page,b,ctx,split", CASES)
def test_plan_edges(dev, orc, Hq, Hkv, d, page, b, ctx, split):  # noqa: F811
    from paper_2607_25852_amd import synth
    R = len(ctx)
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"ranges_h{Hq}_{Hkv}_d{d}_p{page}_R{R}", R=R, b=b,
                              dtype="bf16", Hq=Hq, Hkv=Hkv, d=d, page=page, kv=("list",) + tuple(ctx))
    L = synth.kv_context_lengths(cfg)
    kv = synth.make_kv(cfg, L, fill_unused=np.nan)
    qo = synth.indptr_from_depths(np.array([b - i % b for i in range(R)]))
    say("attn plan", cfg.name, split)
    q, kvl, o, l = run_gpu_attn(dev, cfg, kv, qo, L, kv_split=split)
    check(orc, cfg, kv, qo, kvl, q, o, l)
