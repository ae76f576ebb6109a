"""The inputs of the first-visit tests do what they are for: with the oracle, on the CPU."""
import numpy as np
import pytest

import visit_cases as V
from oracle import mdi_oracle as O
from paper_2505_18164_amd import synth as S
from gpu_util import rel_l2_rows

BAR = 2e-2


def first_visit(cfg, w, x, **changed):
    """The oracle's rows in fp32, with matrices of the first layer replaced."""
    lw = {**w["layers"][0], **changed}
    return O.Partition(cfg, {**w, "layers": {0: lw}}, 0, 1, dtype=np.float32).prefill(0, x)


def moved(cfg, w, x, want, **changed):
    """The share of rows that are beyond the bar with these matrices."""
    return float(np.mean(rel_l2_rows(first_visit(cfg, w, x, **changed), want) > BAR))


def attention_is_seen(cfg, w, x, want=None):
    """Without attention no row meets the bar, and with one that weighs all keys alike none but the first, which has one key."""
    lw = w["layers"][0]
    want = first_visit(cfg, w, x) if want is None else want
    assert rel_l2_rows(first_visit(cfg, w, x, wo=0 * lw["wo"]), want).min() > 5 * BAR
    assert rel_l2_rows(first_visit(cfg, w, x, wq=0 * lw["wq"]), want)[1:].min() > BAR


def no_rotation(rotate):
    return lambda x, positions, base: x


def queries_a_position_further(rotate):
    calls = [0]

    def f(x, positions, base):                             # a layer rotates its queries, then its keys
        calls[0] += 1
        return rotate(x, np.asarray(positions) + calls[0] % 2, base)
    return f


def neighbouring_pairs_swapped(rotate):
    def f(x, positions, base):
        half = np.arange(x.shape[2] // 2) ^ 1
        i = np.concatenate([half, half + x.shape[2] // 2])
        return rotate(x[:, :, i], positions, base)[:, :, i]
    return f


def rotation_is_seen(cfg, w, x, want, monkeypatch, wrong=(no_rotation, queries_a_position_further, neighbouring_pairs_swapped)):
    for f in wrong:
        with monkeypatch.context() as m:
            m.setattr(O, "rope_rotate", f(O.rope_rotate))
            assert moved(cfg, w, x, want) > 0.85, f.__name__


@pytest.mark.parametrize("case", V.HEADS, ids=str)
def test_rotations_matter(case, monkeypatch):
    cfg, w, x = V.heads_visit(*case)
    lw = w["layers"][0]
    want = first_visit(cfg, w, x)
    assert moved(cfg, w, x, want, wo=0 * lw["wo"]) == 1
    if cfg["pos_kind"] == S.POS_ROPE:
        rotation_is_seen(cfg, w, x, want, monkeypatch)
    else:
        assert moved({**cfg, "pos_kind": S.POS_ROPE}, w, x, want) > 0.85


def quick(case):
    _, T, d, heads, kv, h, d_ff, _ = case
    return T * T * heads * h < 1.5e9 and T * d * d_ff < 1.5e9


@pytest.mark.parametrize("case", [c for c in V.TILES if quick(c)], ids=lambda c: str(c[:7]))
def test_every_product_matters(case, monkeypatch):
    cfg, w, x = V.tile_visit(*case)
    lw = w["layers"][0]
    want = first_visit(cfg, w, x)
    down = "wd" if "wd" in lw else "w2"
    assert moved(cfg, w, x, want, wo=0 * lw["wo"]) == 1 and moved(cfg, w, x, want, **{down: 0 * lw[down]}) == 1
    rotation_is_seen(cfg, w, x, want, monkeypatch, (no_rotation,))


# the models a node serves here, with the longest first visit that is measured of each
MODELS = [(S.gpt2_small(), 1024), (S.gpt2_small(dtype=S.DT_F32), 1024), (S.nanollama(), 1024), (S.nanollama(dtype=S.DT_BF16), 2048),
          (S.tinyllama(), 2048), (S.llama2_7b(), 4096), (S.llama3_8b(), 6000)]


def test_every_tile_shape_of_every_product_is_tested():
    needed = set()
    for cfg, longest in MODELS:
        visits = [(cfg, T, most) for T in range(1, longest + 1) for most in {T, cfg["max_ctx"]}]
        needed |= {p for four in V.products(visits) for p in four}
    assert len(needed) > 50
    tested = {p for four in V.products(V.all_visits()) for p in four}
    assert not needed - tested


EVERY_LAUNCH = {(h, g, q) for h in (64, 128) for g, q in ((1, 4), (2, 4), (2, 2), (4, 2))}


@pytest.mark.parametrize("levels", V.LEVELS)
def test_every_launch_of_the_attention_raises_references(levels):
    """... in some queries of a wavefront and not in others, with groups of wavefronts whose references are far apart."""
    raised, mixed, apart = ({k: 0 for k in EVERY_LAUNCH} for _ in range(3))
    for page, heads, kv, h, cuts in V.PAGES:
        cfg, w, x = V.pages_visit(heads, kv, h, cuts, levels)
        s = V.scores_of(cfg, w["layers"][0], x[:sum(cuts)], heads - 1)
        at = 0
        for n in cuts:
            groups, waves = V.launch_of(n, at, heads)
            r, m, a = V.references(s[at:at + n, :at + n], at, n, groups)
            k = (h, groups, waves)
            raised[k], mixed[k], apart[k] = raised[k] + r, mixed[k] + m, max(apart[k], a)
            at += n
    assert min(raised.values()) >= 100 and min(mixed.values()) >= 5
    assert min(a for (_, g, _), a in apart.items() if g > 1) > 10


@pytest.mark.parametrize("T,positions", [(65, 128), (128, 128), (129, 256), (256, 256)])
def test_matrices_beyond_the_fitted_sizes_take_large_tiles(T, positions):
    cfg = S.llama2_7b()
    cfg.update(d_model=8192, n_head=64, n_kv_head=8, d_ff=28672)
    assert V.products([(cfg, T, T)])[0][2] == ("bf16", "swiglu", 256, positions)


@pytest.mark.parametrize("levels", V.LEVELS)
@pytest.mark.parametrize("page,heads,kv,h,cuts", [c for c in V.PAGES if c[1] * c[3] * sum(c[4]) ** 2 < 1.2e9])
def test_attention_matters_in_every_piece(page, heads, kv, h, cuts, levels):
    cfg, w, x = V.pages_visit(heads, kv, h, cuts, levels)
    attention_is_seen(cfg, w, x[:sum(cuts)])


def test_every_launch_of_the_attention_is_reached_with_far_scores():
    assert {(h, *V.launch_of(T, 0, heads)) for heads, _, h, T in V.FAR_VISITS} == EVERY_LAUNCH


@pytest.mark.parametrize("far", V.FAR)
@pytest.mark.parametrize("heads,kv,h,T", V.FAR_VISITS)
def test_far_scores_raise_references_and_matter(heads, kv, h, T, far):
    cfg, w, x = V.far_visit(heads, kv, h, T, far)
    lw = w["layers"][0]
    groups, _ = V.launch_of(T, 0, heads)
    s = V.scores_of(cfg, lw, x, heads - 1)
    raised, _, _ = V.references(s, 0, T, groups)
    assert raised > 100                                    # late queries of sign +1, in every group that sees late keys
    assert s[300:][np.isfinite(s[300:])].min() < -far / 2 and s[300:, 256:][np.isfinite(s[300:, 256:])].max() < 20
    if T < 1000 and far == V.FAR[0]:
        attention_is_seen(cfg, w, x)
