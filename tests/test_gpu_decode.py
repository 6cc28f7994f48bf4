"""Decode steps at the edges of their tiles: appends inside the attention launch, and tile sizes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

METHODS = {
    "fp16": {"method": "fp16"}, "uq": {"method": "uq", "bits": 4, "group": 64},
    "kvq2": {"method": "kvq", "bits": 2, "outlier_bp": 100}, "kvq3": {"method": "kvq", "bits": 3, "outlier_bp": 100},
    "kvq4": {"method": "kvq", "bits": 4, "outlier_bp": 0}, "h2o": {"method": "h2o", "budget_pct": 50},
    "h2o_all": {"method": "h2o", "budget_pct": 100},
}


def _cache(names, lens, hkv, g, d, steps, first=0):
    """A prefilled cache, and the prompt's rows (those of sequence s of a stream that begins at `first`)."""
    import torch
    from paper_2609_07966_amd.cache import KVCache
    rows = []
    for s, n in enumerate(lens):
        r = np.random.default_rng(1000 + first + s)
        rows.append([r.standard_normal((n, h, d)).astype(np.float16) for h in (hkv, hkv, hkv * g)])
    k, v, q = (torch.from_numpy(np.concatenate([x[i] for x in rows])).cuda() for i in range(3))
    r = np.random.default_rng(5)
    books = [float(x) for b in (2, 3, 4) for _ in range(2)
             for x in np.sort(r.uniform(-1, 1, 1 << b)).astype(np.float16)]
    c = KVCache((len(lens), hkv * g, hkv, d, steps), [METHODS[m] for m in names], lens, books)
    c.append_prompt(k, v)
    if any(m.startswith("h2o") for m in names):
        c.h2o_prefill(q)
    return c, rows


def _token(S, hkv, g, d, t):
    import torch
    r = np.random.default_rng(77 + t)
    odd = lambda x: torch.from_numpy(np.concatenate([[0], x.ravel()]).astype(np.float16)).cuda()[1:].view(x.shape)
    return tuple(odd(r.standard_normal((S, h, d))) for h in (hkv, hkv, hkv * g))


@pytest.mark.parametrize("hkv,g,d", [(1, 1, 64), (2, 4, 128), (1, 8, 128), (3, 2, 64)])
def test_step_appends_in_the_attention_launch(hkv, g, d):
    """mkv_decode_step, whose attention launch appends, leaves the same codes, rows, positions, scores
    and outputs as the separate calls, over 70 steps from lengths around the 4-token value
    blocks, the 64-token key blocks and the tile edges (tokens that begin and end a tile)."""
    import torch
    from paper_2609_07966_amd._lib import MkvError
    names = list(METHODS) * 2
    lens = [1, 2, 3, 4, 61, 63, 64, 65, 100, 127, 128, 191, 255, 257]
    S, steps = len(lens), 70
    a, _ = _cache(names, lens, hkv, g, d, steps)
    b, _ = _cache(names, lens, hkv, g, d, steps)
    oa, ob = (torch.full((S, hkv * g, d), float("nan"), device="cuda") for _ in range(2))
    for t in range(steps):
        k, v, q = _token(S, hkv, g, d, t)
        a.step(k, v, q, oa)
        b.append(k, v)
        b.attention(q, ob)
        b.evict()
        # the same tiles in the same order: only the order of atomic additions of value-outlier terms
        # may differ, 128 of them at most a row and each a rounding of 2^-24
        torch.testing.assert_close(oa, ob, rtol=0, atol=float(ob.abs().max()) * 2.0 ** -16, msg=f"step {t}")
        if t % 23 and t != steps - 1:
            continue
        for s, m in enumerate(names):
            for h in range(hkv):
                assert a.counts(s, h) == b.counts(s, h), (t, s, h)
                what = {"f": [], "u": ["codes_k", "codes_v", "scales_k", "scales_v"],
                        "k": ["codes_k", "codes_v", "scales_k", "scales_v", "outliers_k", "outliers_v"],
                        "h": ["positions", "scores"]}[m[0]]
                for w in what:
                    np.testing.assert_array_equal(a.export(s, h, w), b.export(s, h, w), err_msg=f"{w} {m} step {t}")
    with pytest.raises(MkvError):
        a.step(k, v, q, oa)
    a.close()
    b.close()


@pytest.mark.parametrize("name", list(METHODS))
@pytest.mark.parametrize("hkv,g,d", [(2, 4, 128), (1, 2, 64)])
def test_tile_sizes_do_not_change_results(name, hkv, g, d):
    """A launch's tile sizes follow from its sequences: each of these lengths (around the 16-row and
    32-token wave steps and the 64-token tiles) alone, in a batch of its method and beside fp16 rows
    gives the same output up to the rounding of its probabilities; complete fp16 rows also match a float64
    reference."""
    import torch
    lens = [2, 14, 15, 16, 31, 32, 127, 128, 700, 2500]
    S = len(lens)
    k, v, q = _token(2 * S, hkv, g, d, 0)

    def run(names, lens, pick):
        c, rows = _cache(names, lens, hkv, g, d, 1, pick[0])
        out = torch.full((len(lens), hkv * g, d), float("nan"), device="cuda")
        c.step(k[pick].clone(), v[pick].clone(), q[pick].clone(), out)
        c.close()
        return out.cpu().numpy(), rows

    own, rows = run([name] * S, lens, list(range(S)))
    mixed, _ = run([name] * S + ["fp16"] * S, lens + [4000 + 64 * s for s in range(S)], list(range(2 * S)))
    # probabilities (times steps or scales) enter the second product in fp16, relative to a maximum that
    # depends on the tiles: each off by at most 2^-11 of itself (the logits' own roundings add 2^-14 at most)
    # on either side, so an output by that part of the mean of what it weighs: the values' magnitudes, or
    # their distances from the row's minimum under uniform codes.  Where the tokens held or their
    # probabilities are not those of the rows, the largest of these stands for the mean.
    far = []
    for s, (kp, vp, _) in enumerate(rows):
        kk = np.concatenate([kp, k[s:s + 1].cpu().numpy()]).astype(np.float64)
        vv = np.concatenate([vp, v[s:s + 1].cpu().numpy()]).astype(np.float64)
        for e in range(hkv * g):
            x = kk[:, e // g] @ q[s, e].cpu().numpy().astype(np.float64) / np.sqrt(d)
            p = np.exp(x - x.max())
            p /= p.sum()
            vh = vv[:, e // g]
            if name in ("fp16", "h2o_all"):
                far.append((2.0 ** -11 + 2.0 ** -14) * (p @ np.abs(vh)))
                assert (np.abs(own[s, e] - p @ vh) <= far[-1]).all(), (s, e)
            else:
                far.append(np.full(d, (2.0 ** -11 + 2.0 ** -14) * (np.ptp(vh) if name == "uq" else np.abs(vh).max())))
    far = 2 * np.array(far).reshape(S, hkv * g, d)
    assert (np.abs(own - mixed[:S]) <= far).all()
    for s in (0, 3, S - 1):
        alone, _ = run([name], lens[s:s + 1], [s])
        assert (np.abs(alone[0] - own[s]) <= far[s]).all(), s


@pytest.mark.parametrize("name", list(METHODS))
@pytest.mark.parametrize("hkv,g,d", [(2, 4, 128), (1, 2, 64)])
def test_every_token_counts_once(name, hkv, g, d):
    """A query of zeros weighs all tokens alike, and the values of 16 consecutive tokens (a wave's row step)
    share a channel, with those 16 d tokens on (80 tokens at most): one that is lost or taken twice moves an
    output by an 80th of itself or more, the roundings by a 2048th.  The tile sizes of each length alone, of
    the method's batch and beside fp16 rows."""
    import torch
    from oracle import kvquant
    lens = [2, 14, 15, 16, 31, 32, 127, 128, 700, 2500, 4100]
    S, cfg = len(lens), METHODS[name]
    r = np.random.default_rng(5)
    books = {b: [np.sort(r.uniform(-1, 1, 1 << b)).astype(np.float16).astype(np.float32) for _ in range(2)] for b in (2, 3, 4)}

    def onehot(t):
        v = np.zeros((len(t), hkv, d), np.float16)
        v[np.arange(len(t)), :, np.asarray(t) // 16 % d] = 32.0
        return v

    def run(names, lens):
        from paper_2609_07966_amd.cache import KVCache
        n, dev = sum(lens), lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
        k = r.standard_normal((n, hkv, d)).astype(np.float16)
        c = KVCache((len(lens), hkv * g, hkv, d, 1), [METHODS[m] for m in names], lens,
                    [float(x) for b in (2, 3, 4) for half in books[b] for x in half])
        c.append_prompt(dev(k), dev(np.concatenate([onehot(range(m)) for m in lens])))
        held = [np.arange(m) for m in lens]
        if cfg["method"] == "h2o":
            c.h2o_prefill(torch.zeros((sum(m for m, x in zip(lens, names) if x == name), hkv * g, d),
                                      dtype=torch.float16, device="cuda"))
            held = [c.export(s, 0, "positions") for s in range(len(lens))]
        out = torch.full((len(lens), hkv * g, d), float("nan"), device="cuda")
        c.step(dev(r.standard_normal((len(lens), hkv, d)).astype(np.float16)), dev(np.stack([onehot([m])[0] for m in lens])),
               torch.zeros((len(lens), hkv * g, d), dtype=torch.float16, device="cuda"), out)
        c.close()
        return out.cpu().numpy(), held

    def check(out, held, m, where):
        v = onehot(np.append(held, m))[:, 0]
        ref = v.astype(np.float64)
        if cfg["method"] == "kvq":
            cb = books[cfg["bits"]][1]
            code, scale, outl = kvquant.quantize_values(v, cb, cfg["outlier_bp"])
            ref = np.where(outl, ref, cb[code].astype(np.float64) * scale[:, None])
        # equal probabilities are exact; their products with steps or scales round by 2^-11
        assert np.abs(out - ref.mean(axis=0)).max() <= 2.0 ** -11 * np.abs(ref).mean(axis=0).max() + 2.0 ** -20, where

    own = run([name] * S, lens)
    mixed = run([name] * S + ["fp16"] * S, lens + [4000 + 64 * s for s in range(S)])
    for s, m in enumerate(lens):
        check(own[0][s], own[1][s], m, f"{m} tokens")
        check(mixed[0][s], mixed[1][s], m, f"{m} tokens beside others")
        alone = run([name], [m])
        check(alone[0][0], alone[1][0], m, f"{m} tokens alone")


@pytest.mark.parametrize("longest", [1021, 1023, 1500])
@pytest.mark.parametrize("hkv,g,d", [(2, 4, 128), (1, 1, 64)])
def test_selections_with_ties(hkv, g, d, longest):
    """RocketKV steps whose top-k is chosen in the scoring launch (no pair holds over 1024 tokens) and in a
    launch of its own (longest = 1500): the exact top-k of the approximate scores, with keys of
    few values so that equal scores cross the threshold, with all keys equal, and with all kept."""
    import torch
    from oracle import rocketkv
    from paper_2609_07966_amd.cache import KVCache
    lens, topk, nch, steps = [40, 130, 255, 600, 900, longest], [7, 64, 255, 299, 1, 512], 16, 3
    cfgs = [{"method": "rocket", "keep_tokens": 4096, "window": 32, "pool": 7, "topk": t, "n_channels": nch} for t in topk]
    r = np.random.default_rng(d + longest)
    S, at = len(lens), np.concatenate([[0], np.cumsum(lens)])
    k = r.integers(-2, 3, (at[-1], hkv, d)).astype(np.float16)
    k[at[3]:at[4]] = 1.0
    k[at[5]:] = r.standard_normal((longest, hkv, d)).astype(np.float16)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    c = KVCache((S, hkv * g, hkv, d, steps), cfgs, lens)
    c.append_prompt(dev(k), dev(k))
    c.snap_prefill(dev(r.standard_normal((32 * S, hkv * g, d)).astype(np.float16)))
    out = torch.empty((S, hkv * g, d), dtype=torch.float32, device="cuda")
    rows = [k[at[s]:at[s + 1]] for s in range(S)]
    for t in range(steps):
        kn = r.integers(-2, 3, (S, hkv, d)).astype(np.float16)
        q = r.integers(-3, 4, (S, hkv * g, d)).astype(np.float16)
        c.step(dev(kn), dev(kn), dev(q), out)
        for s in range(S):
            rows[s] = np.concatenate([rows[s], kn[s][None]])
            for h in range(hkv):
                hq = q[s, h * g:(h + 1) * g]
                scores = rocketkv.approx_scores(hq, rows[s][:, h], rocketkv.select_channels(hq, nch))
                np.testing.assert_array_equal(c.export(s, h, "topk"), rocketkv.topk_indices(scores, topk[s]),
                                              err_msg=f"sequence {s} head {h} step {t}")
                n = lens[s] + t + 1
                assert c.counts(s, h) == (n, n, min(topk[s], n), lens[s])
    c.close()
