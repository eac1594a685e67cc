"""Row statistics (sv_draft_stats) at row starts and chunk tails of every alignment.

Vocabularies that are no multiple of a 16-byte vector put rows at any element offset, and the
last chunk may hold fewer elements than one vector. Masked logits (-inf and the type's lowest
value), a row of equal values and huge logits take the pass's second path. Bound: each term's
exponent carries a few fp32 roundings of at most |x| log2e < 64 units (2^-24 * 64 * ln 2 per
rounding on a term) and the sum of V positive terms another log2(V) roundings, so 1e-5
relative holds with room; observed values are near 2e-7."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def reference(x, T):
    x = x.astype(np.float64) / T
    m = x.max(axis=1)
    with np.errstate(invalid="ignore"):
        e = np.where(np.isneginf(m)[:, None], 0.0, np.exp(x - np.where(np.isneginf(m), 0.0, m)[:, None]))
    return m, e.sum(axis=1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [1, 3, 7, 8, 9, 4095, 4097, 8191, 8192, 8193, 12289, 50257])
def test_rows_of_every_alignment(V, dtype):
    import torch
    from paper_2607_25852_amd import binding as B
    say("row statistics", V, dtype)
    T = 0.7
    rows = 9
    g = torch.Generator(device="cuda").manual_seed(V)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    x = (torch.randn((rows, V), generator=g, device="cuda") * 4.0).to(dt)
    low = torch.finfo(dt).min
    x[1, : V // 2] = float("-inf")
    x[2, : V // 2] = low
    x[3] = 1.5
    x[4] = low
    x[5] = float("-inf")
    x[6] *= 1e29  # the differences only: every other term underflows
    x[7] += 40.0
    stats = torch.empty((rows, 2), device="cuda")
    conf = torch.empty(rows, device="cuda")
    d = B.draft_stats_desc(1, rows, V, B.SV_F32 if dtype == "f32" else B.SV_BF16, T)
    ws = torch.empty(max(B.draft_stats_workspace_size(d), 256), dtype=torch.uint8, device="cuda")
    B.draft_stats(d, x, stats, conf, ws)
    m, S = reference(x.float().cpu().numpy(), T)
    got = stats.cpu().numpy().astype(np.float64)
    # a row of the lowest value divided by T < 1 overflows fp32: its maximum is -inf, its sum
    # then unspecified but not a wrong finite probability
    ok = np.abs(m) < 3e38
    np.testing.assert_allclose(got[ok, 0], m[ok], rtol=3e-7)
    np.testing.assert_allclose(got[ok, 1], S[ok], rtol=1e-5)
    assert np.isneginf(got[5, 0]) and got[5, 1] == 0.0 and conf[5].item() == 0.0
    np.testing.assert_allclose(conf.cpu().numpy()[ok], 1.0 / S[ok], rtol=1e-5)
