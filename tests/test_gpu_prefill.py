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


@pytest.mark.parametrize("hkv,g,d,bp", [(1, 2, 128, 100), (3, 1, 64, 100), (2, 2, 128, 0), (1, 4, 128, 700), (2, 1, 64, 5000)])
def test_kvq_prompts_at_block_edges(hkv, g, d, bp):
    """Ragged KVQuant prompts of all bit widths quantized together: thresholds, codes, outlier sets and
    value scales bit for bit, with lengths around the 4-token value blocks and the 64-token
    workgroups, outlier-free, one and many value outliers per token, ties and zero tokens, and inputs
    that are aligned to their elements only."""
    import torch
    from oracle import kvquant
    from paper_2609_07966_amd.cache import KVCache
    lens = [1, 2, 4, 7, 63, 64, 65, 130, 257, 300]
    bits = [2 + s % 3 for s in range(len(lens))]
    cfgs = [{"method": "kvq", "bits": b, "outlier_bp": bp} for b in bits]
    r = np.random.default_rng(bp + d)
    n = sum(lens)
    k = (r.standard_normal((n, hkv, d)) * np.exp(r.standard_normal((hkv, d)))).astype(np.float16)
    v = r.standard_normal((n, hkv, d)).astype(np.float16)
    v[::7] = np.round(v[::7])  # many equal magnitudes in a token
    v[5] = 0
    k[::5, :, 3] = k[0, :, 3]
    books, flat = {}, []
    for b in (2, 3, 4):
        half = [np.sort(r.uniform(-1, 1, 1 << b)).astype(np.float16).astype(np.float32) for _ in range(2)]
        books[b] = half
        flat += [float(x) for x in np.concatenate(half)]

    def odd(x):  # on the device, 2 bytes past a 16-byte boundary
        t = torch.empty(x.size + 8, dtype=torch.float16, device="cuda")
        t[1:1 + x.size] = torch.from_numpy(x.reshape(-1)).cuda()
        return t[1:]
    c = KVCache((len(lens), hkv * g, hkv, d, 1), cfgs, lens, codebooks=flat)
    c.append_prompt(odd(k), odd(v))
    at = 0
    for s, (m, b) in enumerate(zip(lens, bits)):
        for h in range(hkv):
            kp, vp = k[at:at + m, h], v[at:at + m, h]
            cbk, cbv = books[b]
            tau, inv = kvquant.calibrate_keys(kp, bp)
            ck, ok = kvquant.quantize_keys(kp, tau, inv, cbk, bp)
            cv, sv, ov = kvquant.quantize_values(vp, cbv, bp)
            where = f"sequence {s} ({m} tokens, {b} bits) head {h}"
            np.testing.assert_array_equal(c.export(s, h, "scales_k"), tau, err_msg=where)
            np.testing.assert_array_equal(c.export(s, h, "codes_k").reshape(m, d), ck, err_msg=where)
            np.testing.assert_array_equal(c.export(s, h, "codes_v").reshape(m, d), cv, err_msg=where)
            np.testing.assert_array_equal(c.export(s, h, "scales_v"), sv, err_msg=where)
            for what, raw, out in (("outliers_k", kp, ok), ("outliers_v", vp, ov)):
                got = c.export(s, h, what).reshape(m, d)
                np.testing.assert_array_equal(got >= 0, out, err_msg=where + what)
                np.testing.assert_array_equal(got[out].astype(np.uint16), raw.view(np.uint16)[out])
            assert c.counts(s, h) == (m, m, m, m)
        at += m
    c.close()


@pytest.mark.parametrize("d,bp", [(128, 100), (64, 5000), (128, 30)])
def test_kvq_thresholds_of_drifting_prompts(d, bp):
    """Thresholds of prompts around the 256-token loads and 512-token batches of the calibration, whose
    magnitudes grow, shrink, stay or alternate along the prompt."""
    import torch
    from oracle import kvquant
    from paper_2609_07966_amd.cache import KVCache
    lens = [255, 257, 511, 512, 513, 1023, 1025, 1500, 2049]
    r = np.random.default_rng(bp)
    k = []
    for n in lens:
        x = np.linspace(-3.0, 3.0, n)[:, None]
        drift = np.stack([x, -x, 0 * x, 3 * np.sign(np.sin(9 * x))])[:, :, 0].T
        k.append((r.standard_normal((n, 1, d)) * np.exp2(drift[:, np.arange(d) % 4])[:, None]).astype(np.float16))
        k[-1][:, :, d // 2:d // 2 + 4] = 1.5
    dev = torch.from_numpy(np.concatenate(k)).cuda()
    cfgs = [{"method": "kvq", "bits": 2, "outlier_bp": bp}] * len(lens)
    books = [float(i) for b in (2, 3, 4) for _ in range(2) for i in range(1 << b)]
    c = KVCache((len(lens), 1, 1, d, 1), cfgs, lens, codebooks=books)
    c.append_prompt(dev, dev)
    for s, n in enumerate(lens):
        np.testing.assert_array_equal(c.export(s, 0, "scales_k"), kvquant.calibrate_keys(k[s][:, 0], bp)[0],
                                      err_msg=f"{n} tokens")
    c.close()


@pytest.mark.parametrize("hkv,g,d,window,pool", [(1, 4, 128, 32, 7), (2, 1, 64, 5, 1), (1, 8, 128, 40, 3), (3, 2, 128, 32, 7)])
def test_snap_prompts_at_chunk_edges(hkv, g, d, window, pool):
    """Ragged RocketKV prompts selected in one launch per stage, some keeping everything: keep-sets
    within the tie band, then one decode step's top-k bit for bit over the gathered keys and their
    channel-major copy, and its output, with lengths around the 32-row and 64-row tiles, the 256-key
    chunks and the 64-slot gathers."""
    import torch
    from gpu_harness import TIE_BAND, TOL, _keep_set_tie_ok
    from oracle import rocketkv, snapkv
    from paper_2609_07966_amd.cache import KVCache
    lens = [41, 64, 65, 255, 257, 300, 511, 513, 700]
    keep = [min(window + 1 + 37 * s, 2 * n) for s, n in enumerate(lens)]
    keep[1], keep[4] = 64, 1000  # the whole prompt
    cfgs = [{"method": "rocket", "keep_tokens": max(t, window), "window": window, "pool": pool, "topk": 0,
             "n_channels": min(d, 32)} for t in keep]
    r = np.random.default_rng(d + window)
    n = sum(lens)
    k = (r.standard_normal((n, hkv, d)) * np.exp(0.5 * r.standard_normal((hkv, d)))).astype(np.float16)
    v = r.standard_normal((n, hkv, d)).astype(np.float16)
    qw = r.standard_normal((window * len(lens), hkv * g, d)).astype(np.float16)
    kn, vn = (r.standard_normal((len(lens), hkv, d)).astype(np.float16) for _ in range(2))
    q = r.standard_normal((len(lens), hkv * g, d)).astype(np.float16)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    c = KVCache((len(lens), hkv * g, hkv, d, 2), cfgs, lens)
    c.append_prompt(dev(k), dev(v))
    c.snap_prefill(dev(qw))
    kept = {(s, h): c.export(s, h, "positions") for s in range(len(lens)) for h in range(hkv)}
    out = torch.empty((len(lens), hkv * g, d), dtype=torch.float32, device="cuda")
    c.step(dev(kn), dev(vn), dev(q), out)
    out = out.cpu().numpy()
    at = 0
    for s, m in enumerate(lens):
        w, T = min(window, m), cfgs[s]["keep_tokens"]
        for h in range(hkv):
            where = f"sequence {s} ({m} tokens, keeping {T}) head {h}"
            hq, kp, vp, pos = slice(h * g, (h + 1) * g), k[at:at + m, h], v[at:at + m, h], kept[s, h]
            if T >= m:
                np.testing.assert_array_equal(pos, np.arange(m), err_msg=where)
            else:
                win = qw[s * window:(s + 1) * window, hq]
                u = snapkv.pooled_votes(win, kp, window, pool)
                ok, _ = _keep_set_tie_ok(np.concatenate([u, np.full(w, np.inf)]), pos,
                                         snapkv.snap_keep(win, kp, T, window, pool), set(range(m - w, m)))
                assert ok, f"keep-set beyond the tie band ({TIE_BAND}): {where}"
            rows_k, rows_v = np.concatenate([kp[pos], kn[s, h][None]]), np.concatenate([vp[pos], vn[s, h][None]])
            ch = rocketkv.select_channels(q[s, hq], cfgs[s]["n_channels"])
            sel = rocketkv.topk_indices(rocketkv.approx_scores(q[s, hq], rows_k, ch), T // 2)
            np.testing.assert_array_equal(c.export(s, h, "topk"), np.append(pos, m)[sel], err_msg=where)
            x = q[s, hq].astype(np.float64) @ rows_k[sel].astype(np.float64).T / np.sqrt(d)
            p = np.exp(x - x.max(axis=1, keepdims=True))
            ref = p / p.sum(axis=1, keepdims=True) @ rows_v[sel].astype(np.float64)
            rms = np.sqrt(np.mean(rows_v[sel].astype(np.float64) ** 2))
            assert np.abs(out[s, hq] - ref).max() <= TOL * rms, where
        at += m
    c.close()


@pytest.mark.parametrize("seqs,longest", [(48, 1100), (30, 1100), (12, 2300)])
def test_snap_prompts_in_long_spans(seqs, longest):
    """Batches that fill the chip take spans of several 128-key steps (of all of a prompt, half of one and
    a quarter here, an odd number of steps among them): keep-sets within the tie band, for prompts that end
    within the first step, at its end and in the last span."""
    import torch
    from gpu_harness import _keep_set_tie_ok
    from oracle import snapkv
    from paper_2609_07966_amd.cache import KVCache
    hkv, g, d, window, pool, keep = 8, 2, 64, 32, 7, 90
    lens = [longest - 17 * s for s in range(seqs)]
    lens[1:4] = 100, 128, 129
    cfgs = [{"method": "rocket", "keep_tokens": keep, "window": window, "pool": pool, "topk": 0, "n_channels": 16}] * seqs
    r = np.random.default_rng(seqs)
    n, at = sum(lens), np.concatenate([[0], np.cumsum(lens)])
    k = r.standard_normal((n, hkv, d)).astype(np.float16)
    qw = r.standard_normal((window * seqs, hkv * g, d)).astype(np.float16)
    dev = lambda x: torch.from_numpy(x).cuda()
    c = KVCache((seqs, hkv * g, hkv, d, 1), cfgs, lens)
    c.append_prompt(dev(k), dev(k))
    c.snap_prefill(dev(qw))
    for s in (0, 1, 2, 3, 4, seqs - 1):
        m = lens[s]
        for h in (0, hkv - 1):
            kp, win = k[at[s]:at[s] + m, h], qw[s * window:(s + 1) * window, h * g:(h + 1) * g]
            u = np.concatenate([snapkv.pooled_votes(win, kp, window, pool), np.full(window, np.inf)])
            ok, _ = _keep_set_tie_ok(u, c.export(s, h, "positions"), snapkv.snap_keep(win, kp, keep, window, pool),
                                     set(range(m - window, m)))
            assert ok, f"sequence {s} ({m} tokens) head {h}"
    c.close()


def test_snap_keep_sets_alone_and_in_a_batch():
    """A sequence keeps the same tokens alone, with a few others (256-key workgroups) and in a batch that
    fills the chip (longer spans).  Two window rows see the same logits in another order, so that their
    sums differ by a rounding at most, and the votes of 40 keys hang on the one, those of 40 others on the
    other: which 60 of them are kept follows the roundings."""
    import torch
    from paper_2609_07966_amd.cache import KVCache
    hkv, g, d, n, seqs = 16, 2, 64, 1024, 24
    cfg = {"method": "rocket", "keep_tokens": 61, "window": 1, "pool": 1, "topk": 0, "n_channels": 8}
    r = np.random.default_rng(7)
    k = np.zeros((seqs, n, hkv, d), np.float16)
    for s in range(seqs):
        for h in range(hkv):
            at = r.permutation(n - 1)
            x = np.minimum(r.standard_normal(n - 81), 2.0)
            k[s, at[:40], h, :2] = 3.0, -3.0
            k[s, at[40:80], h, :2] = -3.0, 3.0
            k[s, at[80:], h, 0], k[s, at[80:], h, 1] = x, r.permutation(x)
    qw = np.zeros((seqs, hkv * g, d), np.float16)
    qw[:, 0::2, 0] = qw[:, 1::2, 1] = 8.0  # the logits are the keys' first two channels
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()

    def kept(which):
        c = KVCache((len(which), hkv * g, hkv, d, 1), [cfg] * len(which), [n] * len(which))
        x = dev(k[which].reshape(-1, hkv, d))
        c.append_prompt(x, x)
        c.snap_prefill(dev(qw[which]))
        got = [[c.export(i, h, "positions") for h in range(hkv)] for i in range(min(3, len(which)))]
        c.close()
        return got

    alone = [kept([s])[0] for s in range(3)]
    for which in ([0, 1, 2], list(range(seqs))):
        np.testing.assert_array_equal(kept(which), alone, err_msg=f"{len(which)} sequences")


@pytest.mark.parametrize("hkv,g,d", [(1, 2, 128), (3, 4, 64), (2, 1, 128)])
def test_uniform_prompts_at_block_edges(hkv, g, d):
    """Ragged uniform 4-bit prompts beside fp16 ones, quantized together: codes and (min, step) pairs bit
    for bit, with lengths around the 4-token value blocks and the 64-token key blocks, constant groups
   ; then a decode step over the incomplete blocks' rows."""
    import torch
    from gpu_harness import TOL
    from oracle import uniform
    from paper_2609_07966_amd.cache import KVCache
    lens = [1, 3, 63, 64, 65, 100, 128, 190, 257]
    cfgs = [{"method": "uq", "bits": 4, "group": 64} if s % 4 else {"method": "fp16"} for s in range(len(lens))]
    r = np.random.default_rng(d + g)
    n, S = sum(lens), len(lens)
    k = (r.standard_normal((n, hkv, d)) * np.exp(r.standard_normal((hkv, d)))).astype(np.float16)
    v = r.standard_normal((n, hkv, d)).astype(np.float16)
    k[:, :, 5] = 0.25
    v[2::9] = -1.5

    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    c = KVCache((S, hkv * g, hkv, d, 1), cfgs, lens)
    c.append_prompt(dev(k), dev(v))
    at = 0
    for s, m in enumerate(lens):
        for h in range(hkv):
            assert c.counts(s, h) == (m, m, m, m)
            if cfgs[s]["method"] != "uq":
                continue
            kp, vp, where = k[at:at + m, h], v[at:at + m, h], f"sequence {s} ({m} tokens) head {h}"
            cv, mn, rng = uniform.quantize_value_rows(vp, 4)
            np.testing.assert_array_equal(c.export(s, h, "codes_v").reshape(m, d), cv, err_msg=where)
            sv = c.export(s, h, "scales_v").reshape(m, d // 64, 2)
            np.testing.assert_array_equal(sv[..., 0], mn, err_msg=where)
            np.testing.assert_array_equal(sv[..., 1], (rng / np.float32(15)).astype(np.float32), err_msg=where)
            nb = m // 64
            gk = c.export(s, h, "codes_k").reshape(-1, d)
            assert gk.shape[0] == 64 * nb
            if nb:
                ck, mn, rng = uniform.quantize_key_blocks(kp, 4)
                np.testing.assert_array_equal(gk, ck, err_msg=where)
                sk = c.export(s, h, "scales_k").reshape(nb, d, 2)
                np.testing.assert_array_equal(sk[..., 0], mn, err_msg=where)
                np.testing.assert_array_equal(sk[..., 1], (rng / np.float32(15)).astype(np.float32), err_msg=where)
        at += m
    kn, vn = (r.standard_normal((S, hkv, d)).astype(np.float16) for _ in range(2))
    q = r.standard_normal((S, hkv * g, d)).astype(np.float16)
    out = torch.empty((S, hkv * g, d), dtype=torch.float32, device="cuda")
    c.step(dev(kn), dev(vn), dev(q), out)
    out = out.cpu().numpy()
    from oracle.sequence import Sequence
    at = 0
    for s, m in enumerate(lens):
        seq = Sequence(cfgs[s], k[at:at + m], v[at:at + m], hkv * g)
        ref, _ = seq.step(kn[s], vn[s], q[s])
        rms = np.sqrt(np.mean(v[at:at + m].astype(np.float64) ** 2))
        assert np.abs(out[s] - ref).max() <= TOL * max(rms, 1.0), f"sequence {s} ({m} tokens)"
        at += m
    c.close()


def test_one_long_prompt_among_short_ones():
    """Batches whose short prompts are prefilled apart from the long one of their method: what a short
    sequence holds is what it holds alone, and its first step attends to its own tokens."""
    import torch
    from gpu_harness import TOL
    from paper_2609_07966_amd.cache import KVCache
    d, longest, short = 64, 60000, 24  # one kv head: groups end at 2^20 idle tokens and twice their own
    methods = [{"method": "fp16"}, {"method": "uq", "bits": 4, "group": 64}, {"method": "kvq", "bits": 3, "outlier_bp": 100},
               {"method": "h2o", "budget_pct": 50},
               {"method": "rocket", "keep_tokens": 60, "window": 16, "pool": 3, "topk": 0, "n_channels": 8}]
    cfgs, lens = [], []
    for s in range(short + 1):
        cfgs += methods
        lens += [longest if s == 7 else 90 + 3 * s] * len(methods)
    n, S, at = sum(lens), len(lens), np.concatenate([[0], np.cumsum(lens)])
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *shape: torch.randn(shape, generator=g, device="cuda").half()
    k, v, kn, vn, q, qw = rand(n, 1, d), rand(n, 1, d), rand(S, 1, d), rand(S, 1, d), rand(S, 1, d), rand(S, 16, 1, d)
    books = [float(i) / 16 - 0.5 for b in (2, 3, 4) for _ in range(2) for i in range(1 << b)]

    def admit(which):
        c = KVCache((len(which), 1, 1, d, 1), [cfgs[s] for s in which], [lens[s] for s in which], codebooks=books)
        rows = lambda x: torch.cat([x[at[s]:at[s + 1]] for s in which])
        c.append_prompt(rows(k), rows(v))
        of = lambda m: [s for s in which if cfgs[s]["method"] == m]
        if of("h2o"):
            c.h2o_prefill(torch.cat([k[at[s]:at[s + 1]] for s in of("h2o")]))  # (queries equal to the keys)
        if of("rocket"):
            c.snap_prefill(qw[of("rocket")].contiguous())
        held = lambda i, s: [c.export(i, 0, what) for what in
                             {"fp16": ["counts"], "uq": ["codes_k", "codes_v", "scales_v"],
                              "kvq": ["codes_k", "codes_v", "outliers_k", "scales_k"],
                              "h2o": ["positions", "scores"], "rocket": ["positions"]}[cfgs[s]["method"]]]
        out = torch.empty((len(which), 1, d), dtype=torch.float32, device="cuda")
        got = [held(i, s) for i, s in enumerate(which)]
        c.step(kn[which].contiguous(), vn[which].contiguous(), q[which].contiguous(), out)
        out = out.cpu().numpy()
        c.close()
        return got, out

    batch, out = admit(list(range(S)))
    for s in list(range(0, 10)) + list(range(S - 10, S)):
        alone, ref = admit([s])
        for a, b in zip(batch[s], alone[0]):
            np.testing.assert_array_equal(a, b, err_msg=f"sequence {s}: {cfgs[s]}")
        assert np.abs(out[s] - ref[0]).max() <= TOL, f"sequence {s}: {cfgs[s]}"
