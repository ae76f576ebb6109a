"""The inputs of the first-visit tests do what they are for: with the float64 oracle, on the CPU."""
import numpy as np
import pytest

import visit_cases as V
from oracle import mdi_oracle as O
from gpu_util import rel_l2_rows

BAR = 2e-2


def first_visit(cfg, w, x, **changed):
    """The oracle's rows, with matrices of the first layer replaced."""
    lw = {**w["layers"][0], **changed}
    return O.Partition(cfg, {**w, "layers": {0: lw}}, 0, 1).prefill(0, x)


def seen_in_all_rows(cfg, w, x, want=None):
    """Without attention, and with one that weighs all keys alike, no row (but the first, which has one key) meets the bar."""
    lw = w["layers"][0]
    want = first_visit(cfg, w, x) if want is None else want
    assert rel_l2_rows(first_visit(cfg, w, x, wo=0 * lw["wo"]), want).min() > 5 * BAR
    assert rel_l2_rows(first_visit(cfg, w, x, wq=0 * lw["wq"]), want)[1:].min() > BAR


@pytest.mark.parametrize("far", V.FAR)
@pytest.mark.parametrize("heads,kv,h,T", V.FAR_VISITS)
def test_far_scores_raise_references_and_matter(heads, kv, h, T, far):
    cfg, w, x = V.far_visit(heads, kv, h, T, far)
    lw = w["layers"][0]
    groups, _ = V.launch_of(T, 0, heads)
    for head in (0, heads - 1):
        s = V.scores_of(cfg, lw, x, head)
        raised, _, _ = V.references(s, 0, T, groups)
        assert raised > 100                                # late queries of sign +1, once per group of wavefronts that sees late keys
        assert s[300:][np.isfinite(s[300:])].min() < -far / 2 and s[300:, 256:][np.isfinite(s[300:, 256:])].max() < 20
    seen_in_all_rows(cfg, w, x)


def test_every_launch_of_the_attention_is_reached_with_far_scores():
    assert {(h, *V.launch_of(T, 0, heads)) for heads, _, h, T in V.FAR_VISITS} == {(h, g, q) for h in (64, 128) for g, q in ((1, 4), (2, 4), (2, 2), (4, 2))}
