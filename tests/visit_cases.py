"""Inputs of the first-visit tests whose results depend on what is tested: attention that moves every row, scores that are
far apart, rotations that matter.  CPU only (numpy); tests/test_visit_cases.py asserts that they do what they are for."""
import math

import numpy as np

from oracle import mdi_oracle as O
from paper_2505_18164_amd import synth as S

BK, RAISE = 64, 8.0          # keys of a block; powers of two a score may exceed its query's reference (attn_prefill.hip)

def loud(cfg, w, scores=1.4, attention=3.0, mlp=1.0):
    """Scales the matrices by their inner dimensions, so that every one of them moves the result: scores of about
    N(0, scores^2), an attention output of up to `attention` and an MLP output of about `mlp` times a row of N(0, 1)."""
    d, H, h, F = cfg["d_model"], cfg["n_head"], cfg["head_dim"], cfg["d_ff"]
    gain = dict(wq=math.sqrt(scores / d), wk=math.sqrt(scores / d), wv=1 / math.sqrt(d), wo=attention / math.sqrt(H * h),
                w1=1 / math.sqrt(d), w2=mlp * 2 / math.sqrt(F), wg=1 / math.sqrt(d), wu=1 / math.sqrt(d), wd=mlp * 2 / math.sqrt(F))
    for lw in w["layers"].values():
        for name, k in gain.items():
            if name in lw:
                lw[name] = S.storage_round(lw[name] * np.float32(k / S.WEIGHT_STD), cfg["dtype"])
    return w


# Channels of a marked row (every entry +1 or -1, so that its norm is exactly 1): 0 - 7 the key's level n in binary, 8 always
# +1, 9 and 10 the query's sign (their mean), 11 -1 where the key is far away
_LEVEL, _ONE, _SIGN, _FAR = 8, 8, 9, 11


def marked_cfg(heads, kv, h, max_ctx):
    c = S.tiny(n_layer=1, d_model=64, n_head=heads, n_kv_head=kv, head_dim=h, d_ff=96, vocab=61, max_ctx=max_ctx, dtype=S.DT_BF16,
               pos_kind=S.POS_LEARNED)
    c["norm_eps"] = 0.0
    return c


def marked_weights(cfg, seed, rise=0.0, far=0.0):
    """Channel 0 of a head's queries and keys carries levels that are exact in bf16, the others random content (scores of
    about N(0, 1.4^2)).  A key's level n adds `rise` n powers of two to the score of a query with sign +1 (even heads; odd
    heads: sign -1), far keys subtract `far` powers of two.  The attention's part of a row is about as large as the row."""
    H, K, h, d = cfg["n_head"], cfg["n_kv_head"], cfg["head_dim"], cfg["d_model"]
    assert d == 64 and not (rise and far)
    g = np.random.Generator(np.random.PCG64([seed, H, h]))
    w = S.make_weights(cfg, seed)
    lw = w["layers"][0]
    wq, wk = (g.standard_normal((n, h, d)) * 1.2 / math.sqrt(d) for n in (H, K))
    wq[:, 0, :] = wk[:, 0, :] = 0.0
    unit = math.sqrt(h) / math.log2(math.e)                          # a product of q and k that is worth one power of two
    q0, k_scale = (rise * unit / 2, 1.0) if rise else (math.sqrt(far * unit), math.sqrt(far * unit))
    if rise:
        wk[:, 0, :_LEVEL] = 2.0 ** np.arange(_LEVEL)                 # 2 n - 255
        wk[:, 0, _ONE] = 255.0
    elif far:
        k_scale = 2.0 ** round(math.log2(k_scale))
        q0 = far * unit / k_scale
        wk[:, 0, _ONE], wk[:, 0, _FAR] = -k_scale / 2, k_scale / 2   # 0 or -k_scale
    sign = np.where(np.arange(H) % 2 == 0, 1.0, -1.0) if rise else np.ones(H)
    wq[:, 0, _SIGN] = wq[:, 0, _SIGN + 1] = (sign * q0 / 2)
    lw["wq"], lw["wk"] = (S.round_to_bf16(m.reshape(-1, d).astype(np.float32)) for m in (wq, wk))
    lw["wv"] = S.round_to_bf16((g.standard_normal((K * h, d)) / math.sqrt(d)).astype(np.float32))
    lw["wo"] = S.round_to_bf16((g.standard_normal((d, H * h)) * 2 / math.sqrt(H * h)).astype(np.float32))
    return w


def marked_rows(T, seed, run=16, levels="up", far_keys=0):
    """T rows.  Positions in runs of `run` share a level: n = 0, 1, 2, ... ("up") or any of 0 .. 255 ("any").  The first
    `far_keys` positions are far away as keys and have sign 0 as queries."""
    g = np.random.Generator(np.random.PCG64([seed, T, run, far_keys]))
    x = np.where(g.random((T, 64)) < 0.5, -1.0, 1.0).astype(np.float32)
    runs = (T + run - 1) // run
    n = np.arange(runs) if levels == "up" else g.integers(0, 256, runs)
    assert n.max() < 256
    n = np.repeat(n, run)[:T]
    x[:, :_LEVEL] = np.where((n[:, None] >> np.arange(_LEVEL)) & 1, 1.0, -1.0)
    x[:, _ONE] = 1.0
    x[:, _FAR] = 1.0
    if far_keys:
        x[:, _SIGN] = 1.0                                            # signs 0 and +1 only: nothing else is left of a score of -2^26
        x[:far_keys, _FAR] = -1.0
        x[:far_keys, _SIGN + 1] = -1.0
    return x


def launch_of(T, p0, H):
    """(groups, wavefronts per group) of the attention launch for T positions behind p0 (launch_flash_heads)."""
    items = -(-T // 128) * H
    if items >= 384 or p0 + T <= BK:
        return 1, 4
    if items > 128:
        return 2, 4
    return (4, 2) if p0 + T // 2 >= 320 else (2, 2)


def scores_of(cfg, lw, x, head):
    """Scores of one head in powers of two [T, T], hidden ones -inf (rows of the first layer, no rotation)."""
    H, K, h = cfg["n_head"], cfg["n_kv_head"], cfg["head_dim"]
    a = O._norm(cfg, np.asarray(x, np.float64), lw["ln1_g"].astype(np.float64), None)
    q = a @ lw["wq"].astype(np.float64)[head * h:(head + 1) * h].T
    kvh = head // (H // K)
    k = a @ lw["wk"].astype(np.float64)[kvh * h:(kvh + 1) * h].T
    s = q @ k.T * (math.log2(math.e) / math.sqrt(h))
    return np.where(np.tri(len(x), dtype=bool), s, -np.inf)


def references(s, p0, T, groups):
    """Follows every query's reference through the blocks of its group: the maximum of the first block, raised where a
    score of the wavefront's 32 queries exceeds it by more than 2^8.  s: [queries p0 .. p0 + T - 1, keys].  Returns (raises of
    queries, raises that left other queries of the wavefront alone, largest difference between two groups of a query)."""
    n_kb = -(-s.shape[1] // BK)
    pad = np.full((T, n_kb * BK - s.shape[1]), -np.inf)
    tops = np.concatenate([s, pad], axis=1).reshape(T, n_kb, BK).max(axis=2)
    raised = mixed = 0
    refs = []
    for g in range(groups):
        ref = np.full(T, -np.inf)
        for kb in range(g, n_kb, groups):
            for w in range(0, T, 32):
                r, t = ref[w:w + 32], tops[w:w + 32, kb]
                if not np.any(t > -np.inf):
                    continue
                if np.all(r == -np.inf):
                    ref[w:w + 32] = t
                elif np.any(t > r + RAISE):
                    raised += int(np.sum(t > r + RAISE))
                    mixed += int(np.any(t <= r))
                    ref[w:w + 32] = np.maximum(r, t)
        refs.append(ref)
    refs = np.stack(refs)
    seen = refs > -np.inf
    both = seen.sum(axis=0) > 1
    apart = (np.where(seen, refs, -np.inf).max(axis=0) - np.where(seen, refs, np.inf).min(axis=0))[both]
    return raised, mixed, float(apart.max()) if both.any() else 0.0


# First visits whose late keys lie 2^26 or 2^120 powers of two above the first 256: a launch of every kind for both head sizes
FAR = (2.0 ** 26, 2.0 ** 120)
FAR_VISITS = [(heads, kv, h, T) for h in (64, 128) for heads, kv, T in ((32, 4, 1600), (32, 8, 704), (4, 2, 600), (8, 2, 704))]


def far_visit(heads, kv, h, T, far):
    cfg = marked_cfg(heads, kv, h, T)
    return cfg, marked_weights(cfg, 80, far=far), marked_rows(T, 81, far_keys=256)
