"""Prefill kernels at the edges of their tiles, against plain references."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _causal_scores(q, k):
    """float64: attention received by every token, summed over rows and query heads.  q [n][G][d], k [n][d]."""
    n, _, d = q.shape
    s = np.einsum("igd,jd->gij", q.astype(np.float64), k.astype(np.float64)) / np.sqrt(d)
    s[:, np.triu(np.ones((n, n), bool), 1)] = -np.inf
    s -= s.max(axis=2, keepdims=True)
    p = np.exp(s)
    return (p / p.sum(axis=2, keepdims=True)).sum(axis=(0, 1)), s


@pytest.mark.parametrize("hkv,g,d", [(1, 1, 128), (2, 2, 64), (3, 4, 128), (1, 8, 128), (2, 8, 64)])
def test_h2o_scores_at_tile_edges(hkv, g, d):
    """Ragged prompts around the 32-key subtiles, 64-item stages, 256-item blocks and the shortest row
    segment, scored in one launch; the last two sequences' logits grow by hundreds of powers of two
    along the prompt, so that rows leave the reference of their first tile."""
    import torch
    from paper_2609_07966_amd.cache import KVCache
    lens = [1, 5, 31, 33, 64, 65, 127, 255, 257, 300, 513, 300, 200]
    cfgs = [{"method": "h2o", "budget_pct": 100}] * len(lens)
    r = np.random.default_rng(d + g)
    k = r.standard_normal((sum(lens), hkv, d)).astype(np.float16)
    v = r.standard_normal((sum(lens), hkv, d)).astype(np.float16)
    q = r.standard_normal((sum(lens), hkv * g, d)).astype(np.float16)
    at = np.concatenate([[0], np.cumsum(lens)])
    for s in (len(lens) - 2, len(lens) - 1):
        ramp = np.exp2(np.linspace(0.0, 6.0, lens[s]))[:, None, None]
        k[at[s]:at[s + 1]] = (k[at[s]:at[s + 1]] * ramp).astype(np.float16)
        q[at[s]:at[s + 1]] = (q[at[s]:at[s + 1]] * 4).astype(np.float16)
    c = KVCache((len(lens), hkv * g, hkv, d, 1), cfgs, lens)
    c.append_prompt(torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda())
    c.h2o_prefill(torch.from_numpy(q).cuda())
    for s, n in enumerate(lens):
        for h in range(hkv):
            a, b = at[s], at[s + 1]
            ref, logits = _causal_scores(q[a:b, h * g:(h + 1) * g], k[a:b, h])
            np.testing.assert_array_equal(c.export(s, h, "positions"), np.arange(n))
            got = c.export(s, h, "scores")
            # a logit x is off by at most |x| 2^-24 per rounding, and by d 2^-24 of the sum of its
            # products' magnitudes from the matrix core (under 2 |x|max here); the row's sum likewise
            x = np.abs(np.where(np.isfinite(logits), logits, 0)).max() + 8
            np.testing.assert_allclose(got, ref, rtol=0, atol=float((6 * x + n) * 2.0 ** -23) * max(1.0, ref.max()),
                                       err_msg=f"sequence {s} (n = {n}) head {h}")
    c.close()
