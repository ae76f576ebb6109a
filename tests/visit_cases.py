"""Inputs of the first-visit tests whose results depend on what is tested: attention that moves every row, scores that are
far apart, rotations that matter.  CPU only (numpy); tests/test_visit_cases.py asserts that they do what they are for."""
import functools
import math
import os
import subprocess
import tempfile

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


@functools.lru_cache(None)
def launch_of(T, p0, H):
    """(groups, wavefronts per group) of the attention launch for T positions behind p0."""
    return tuple(int(v) for v in _ask(["-1 0 %d 0 0 0 0 %d %d" % (H, T, p0)])[0].split())


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


F32 = dict(dtype=S.DT_F32)
GELU = dict(norm_kind=S.NORM_LAYERNORM, mlp_kind=S.MLP_GELU_TANH, has_bias=1)


def ragged(**kw):
    base = dict(n_layer=1, d_model=520, n_head=8, n_kv_head=4, head_dim=64, d_ff=4104, vocab=61, max_ctx=2304, dtype=S.DT_BF16)
    base.update(kw)
    return S.tiny(**base)


EDGES = [(T, {}) for T in (1, 31, 32, 33, 64, 65, 130, 257, 700, 2050)] + [(T, GELU) for T in (16, 129, 515)] \
    + [(T, F32) for T in (1, 32, 33, 64, 65, 200, 700)] + [(T, dict(GELU, **F32)) for T in (31, 300)]

# storage type, T, d, heads, kv heads, head size, d_ff, MLP: every tile shape in every product that the models of synth.py take
# it for and more, none of the sizes a multiple of its tiles
TILES = [(S.DT_BF16, *v) for v in (
    (9, 72, 2, 2, 64, 24, GELU), (1300, 3080, 2, 2, 64, 520, GELU), (1300, 1032, 2, 2, 64, 6152, GELU), (2050, 72, 32, 8, 64, 2056, GELU),
    (3000, 3080, 2, 2, 64, 2056, GELU), (2050, 72, 2, 2, 64, 6152, GELU), (700, 3080, 64, 32, 128, 24, GELU), (2050, 6152, 2, 2, 64, 24, GELU),
    # 256 x 256, 256 x 192
    (2090, 72, 32, 32, 64, 2056, GELU), (1473, 72, 2, 2, 64, 4104, {}),
    (1068, 72, 32, 32, 64, 2056, GELU), (973, 3080, 8, 2, 64, 5512, GELU), (1971, 3080, 2, 1, 64, 24, GELU), (1199, 72, 2, 2, 64, 5144, GELU),
    # 192 x 192, 128 x 192
    (1408, 1032, 32, 32, 64, 24, GELU), (1182, 3208, 4, 1, 64, 4104, {}), (2475, 3080, 16, 2, 64, 24, {}), (688, 1032, 4, 4, 64, 5656, {}),
    (543, 72, 32, 32, 64, 5360, GELU), (328, 3080, 64, 2, 64, 24, GELU), (1195, 3080, 2, 1, 64, 24, GELU), (394, 72, 2, 2, 64, 4104, {}),
    # 96 x 128, 64 x 96
    (400, 72, 32, 32, 64, 24, GELU), (2092, 1032, 2, 1, 64, 4104, GELU), (195, 72, 2, 1, 64, 4104, {}),
    (70, 72, 16, 4, 64, 24, GELU), (267, 1032, 2, 2, 64, 24, GELU), (83, 72, 4, 2, 64, 2056, {}),
    # QKV on 192 x 128, 256 x 128, 192 x 256; residual on 192 x 128, 256 x 128; split on 128 x 128, 192 x 128, 256 x 128, 256 x 256
    (393, 72, 64, 16, 128, 24, GELU), (577, 72, 64, 8, 128, 24, {}), (962, 24, 64, 16, 128, 72, {}), (1355, 4104, 1, 1, 64, 24, {}),
    (1457, 4104, 4, 1, 64, 24, {}), (194, 3080, 1, 1, 128, 4104, GELU), (195, 4104, 64, 8, 64, 24, {}), (193, 5128, 1, 1, 64, 14344, GELU),
    (385, 3080, 1, 1, 64, 14344, GELU),
    # up on 128 x 64, 128 x 128; gate/up on 128 x 128, 192 x 128, 192 x 256
    (133, 24, 1, 1, 128, 6152, GELU), (305, 24, 2, 2, 64, 8200, GELU), (193, 24, 2, 1, 64, 6152, {}), (195, 24, 1, 1, 64, 8200, {}), (991, 24, 2, 2, 64, 5624, {}))]
TILES += [(S.DT_F32, *v) for v in ((300, 520, 24, 8, 64, 72, GELU), (257, 3080, 2, 2, 64, 72, GELU), (700, 2056, 2, 2, 64, 1032, GELU), (700, 2056, 2, 2, 64, 520, {}))]


def tile_cfg(dtype, T, d, heads, kv, h, d_ff, mlp):
    return S.tiny(n_layer=1, d_model=d, n_head=heads, n_kv_head=kv, head_dim=h, d_ff=d_ff, vocab=61, max_ctx=T, **{**mlp, "dtype": dtype})


def tile_visit(*case):
    cfg = tile_cfg(*case)
    return cfg, loud(cfg, S.make_weights(cfg, 55, exercise=True)), S.make_activations(cfg, 56, 0, case[1])


# T, d, head size, heads, kv heads, options: a first piece of T positions and a second of 20
HEADS = [
    (1408, 1032, 256, 8, 8, {}), (1408, 1032, 128, 16, 16, GELU), (400, 72, 256, 8, 8, {}), (400, 72, 128, 16, 16, {}),
    (333, 520, 128, 9, 3, {}), (37, 72, 256, 3, 1, GELU), (333, 72, 8, 6, 3, {}), (65, 520, 16, 12, 2, dict(GELU, pos_kind=S.POS_LEARNED)),
    (130, 72, 32, 5, 5, dict(pos_kind=S.POS_LEARNED)), (65, 72, 256, 3, 3, F32), (100, 520, 64, 10, 2, F32), (33, 72, 8, 4, 2, dict(GELU, **F32))]


def heads_cfg(T, d, h, heads, kv, kw):
    return S.tiny(n_layer=1, d_model=d, n_head=heads, n_kv_head=kv, head_dim=h, d_ff=72, vocab=61, max_ctx=T + 21, **{"dtype": S.DT_BF16, **kw})


def heads_visit(T, *case):
    cfg = heads_cfg(T, *case)
    return cfg, loud(cfg, S.make_weights(cfg, 64, exercise=True)), S.make_activations(cfg, 65, 0, T + 20)


# positions per page, heads, kv heads, head size, pieces
PAGES = [(64, 4, 2, 128, (130, 62, 1, 200)), (128, 4, 4, 64, (1, 127, 129, 64)), (48, 4, 1, 128, (100, 93, 7)),
         (16, 4, 2, 64, (15, 17, 96, 200)), (5, 2, 2, 64, (64, 70)), (64, 32, 8, 64, (1600,)),
         (24, 32, 4, 128, (1540, 3)),
         # around the rule between 64 and 128 queries per workgroup (128 items of 128 queries)
         (64, 16, 4, 128, (1024, 65, 1)), (64, 16, 4, 128, (1025, 63)), (24, 16, 8, 64, (1089, 95)), (64, 8, 8, 128, (1, 31, 33, 64, 66)),
         # ... and between two and four groups (320 keys on average)
         (64, 8, 2, 128, (639, 1, 64, 65)), (16, 8, 8, 64, (319, 2, 1, 200)), (64, 8, 8, 128, (640,)), (128, 8, 4, 64, (700, 33))]
LEVELS = {"up": 3.0, "any": 1.0}     # powers of two per level


def pages_visit(heads, kv, h, cuts, levels):
    T = sum(cuts)
    cfg = marked_cfg(heads, kv, h, 1664)
    return cfg, marked_weights(cfg, 70, rise=LEVELS[levels]), marked_rows(T + 1, 71, levels=levels)


# First visits whose late keys lie 2^26 or 2^120 powers of two above the first 256: a launch of every kind for both head sizes
FAR = (2.0 ** 26, 2.0 ** 120)
FAR_VISITS = [(heads, kv, h, T) for h in (64, 128) for heads, kv, T in ((32, 4, 1600), (32, 8, 704), (4, 2, 600), (8, 2, 704))]


def far_visit(heads, kv, h, T, far):
    cfg = marked_cfg(heads, kv, h, T)
    return cfg, marked_weights(cfg, 80, far=far), marked_rows(T, 81, far_keys=256)


def dominated_visit():
    """Queries whose weight lies on one key or a few, with references up to 2^8 below it."""
    cfg = marked_cfg(32, 8, 128, 1600)
    return cfg, marked_weights(cfg, 70, rise=12.0), marked_rows(1600, 71, run=1, levels="any")


# ----------------------------------------------------------------------------
# Which kernels a first visit's products run on, asked of the plan itself (csrc/visit_plan.h)
_PLAN = r"""
#include <cstdio>
#include <algorithm>
#include "visit_plan.h"
int main() {
  int dtype, d, H, K, h, F, swiglu, T, Tm;
  while (std::scanf("%d %d %d %d %d %d %d %d %d", &dtype, &d, &H, &K, &h, &F, &swiglu, &T, &Tm) == 9) {
    if (dtype < 0) {
      const mdi::FlashPlan p = mdi::plan_flash(T, Tm, H);
      std::printf("%d %d\n", p.groups, p.waves);
      continue;
    }
    const size_t cap = std::min<size_t>((size_t)Tm * mdi::kMaxKSplits, 4096) * d;
    const mdi::GemmPlan p[4] = {mdi::plan_gemm(dtype, 256, T, (H + 2 * K) * h, d, 0), mdi::plan_gemm(dtype, 256, T, d, H * h, cap),
                                mdi::plan_gemm(dtype, 256, T, swiglu ? 2 * F : F, d, 0), mdi::plan_gemm(dtype, 256, T, d, F, cap)};
    for (const auto& q : p) {
      const mdi::Shape& s = dtype == MDI_BF16 ? mdi::kShapesBf16[q.shape] : mdi::kShapesF32[q.shape];
      std::printf("%d %d %d ", s.BN, s.BT, q.S);
    }
    std::printf("\n");
  }
}
"""


@functools.lru_cache(None)
def _plan_program():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    d = _plan_program.dir.name
    src, exe = os.path.join(d, "plan.cpp"), os.path.join(d, "plan")
    open(src, "w").write(_PLAN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(root, "paper_2505_18164_amd", "csrc"), "-I", os.path.join(root, "include"), src, "-o", exe],
                   check=True)
    return exe


_plan_program.dir = tempfile.TemporaryDirectory()


def _ask(lines):
    return subprocess.run([_plan_program()], input="\n".join(lines) + "\n", check=True, capture_output=True, text=True).stdout.splitlines()


def products(visits):
    """Of every (cfg, T, max_prefill): what its four products run on, as (dtype, epilogue, rows, positions of a tile)."""
    lines = []
    for c, T, Tm in visits:
        lines.append("%d %d %d %d %d %d %d %d %d" % (c["dtype"], c["d_model"], c["n_head"], c["n_kv_head"], c["head_dim"], c["d_ff"],
                                                     c["mlp_kind"] == S.MLP_SWIGLU, T, Tm))
    res = []
    for (c, _, _), line in zip(visits, _ask(lines)):
        v = [int(x) for x in line.split()]
        mlp = "swiglu" if c["mlp_kind"] == S.MLP_SWIGLU else "gelu"
        dt = "bf16" if c["dtype"] == S.DT_BF16 else "f32"
        kinds = ["qkv", "split" if v[5] > 1 else "resid", mlp, "split" if v[11] > 1 else "resid"]
        res.append([(dt, k, v[3 * i], v[3 * i + 1]) for i, k in enumerate(kinds)])
    return res


def all_visits():
    """Every first visit that the tests compare with the oracle, as products takes it."""
    v = [(ragged(**kw), T, T) for T, kw in EDGES] + [(tile_cfg(*c), c[1], c[1]) for c in TILES]
    v += [(heads_cfg(*c), t, c[0]) for c in HEADS for t in (c[0], 20)]
    v += [(marked_cfg(heads, kv, h, 1664), n, max(cuts)) for _, heads, kv, h, cuts in PAGES for n in cuts]
    return v + [(marked_cfg(heads, kv, h, T), T, T) for heads, kv, h, T in FAR_VISITS]
