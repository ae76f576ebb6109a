"""The shared pass with workgroups of four and of eight wavefronts: column slices that do not divide evenly, wavefronts without
columns, blocks past the last, slices of an inner dimension that one round of requests does not cover, slices of two weight
tiles next to slices of one, and passes that change from one kind of workgroup to the other."""
import numpy as np
import pytest

from paper_2505_18164_amd import synth as S
from gpu_util import check, dev_ids, pair, scale_matrices

pytestmark = pytest.mark.gpu

SHAPES = {
    "17 column steps": dict(d_model=544, n_head=17, n_kv_head=17, head_dim=32, d_ff=1056),
    "one column step": dict(d_model=32, n_head=2, n_kv_head=1, head_dim=16, d_ff=32, norm_kind=S.NORM_LAYERNORM, mlp_kind=S.MLP_GELU_TANH, has_bias=1),
    "9 column steps, LayerNorm": dict(d_model=288, n_head=9, n_kv_head=3, head_dim=32, d_ff=608, norm_kind=S.NORM_LAYERNORM, mlp_kind=S.MLP_GELU_ERF,
                                      pos_kind=S.POS_LEARNED, has_bias=1),
    "long slices": dict(d_model=256, n_head=4, n_kv_head=2, head_dim=64, d_ff=12288, mlp_kind=S.MLP_GELU_TANH),
    "more blocks than workgroups": dict(d_model=64, n_head=4, n_kv_head=2, head_dim=16, d_ff=5152),
    # more than eight steps to a wavefront are two tiles: with four wavefronts slices of 9, 9, 9 and 8 steps, and of 16, 16, 16
    # and 15; with eight (four cannot hold this width) seven of 10 and one of 3
    "35 column steps": dict(d_model=1120, n_head=4, n_kv_head=2, head_dim=32, d_ff=160),
    "35 column steps, LayerNorm": dict(d_model=1120, n_head=4, n_kv_head=2, head_dim=32, d_ff=160, norm_kind=S.NORM_LAYERNORM, mlp_kind=S.MLP_GELU_TANH, has_bias=1),
    "63 column steps": dict(d_model=2016, n_head=4, n_kv_head=1, head_dim=32, d_ff=96, mlp_kind=S.MLP_GELU_ERF),
    "63 column steps, LayerNorm": dict(d_model=2016, n_head=4, n_kv_head=1, head_dim=32, d_ff=96, norm_kind=S.NORM_LAYERNORM),
    "73 column steps": dict(d_model=2336, n_head=4, n_kv_head=1, head_dim=32, d_ff=96),
    "73 column steps, LayerNorm": dict(d_model=2336, n_head=4, n_kv_head=1, head_dim=32, d_ff=96, norm_kind=S.NORM_LAYERNORM, mlp_kind=S.MLP_GELU_TANH, has_bias=1),
}


@pytest.mark.parametrize("n_msg", [3, 16])
@pytest.mark.parametrize("waves", ["4", "8"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_shared_pass(name, waves, n_msg, monkeypatch):
    monkeypatch.setenv("MDI_BATCH_WAVES", waves)
    cfg = S.tiny(n_layer=2, dtype=S.DT_BF16, max_ctx=64, vocab=97, **SHAPES[name])
    # Matrices such that products of a normalised vector have the same variance at every width past the first shape's: wide
    # vectors times 2 make scores so large that the softmax amplifies bf16 rounding (2016 columns, LayerNorm: up to 2.1e-2
    # here and 1.9e-2 from one message at a time; like this 1.1e-2 and 9e-3).
    scale = min(2.0, 2.0 * (544 / cfg["d_model"]) ** 0.5) if cfg["d_ff"] < 4096 else 1.0
    w = scale_matrices(S.make_weights(cfg, 41, exercise=True), scale)
    o, g = pair(cfg, w, 0, 2, embed=True, head=False, max_seqs=n_msg, kv_page_tokens=8)
    assert g.info(4) == 16
    for s, ids in enumerate(S.make_prompts(cfg, 41, n_msg, 7)):
        check(g.prefill(s, dev_ids(ids)), o.prefill(s, ids), cfg, ("prefill", s))
    rng = np.random.default_rng(9)
    order = list(range(n_msg))
    for step in range(3):
        toks = [int(rng.integers(0, cfg["vocab"])) for _ in order]
        for s, t, got in zip(order, toks, g.decode_batch(order, [dev_ids([t]) for t in toks])):
            check(got, o.decode_step(s, t), cfg, ("batched decode", step, s))
    assert g.info(7) == (8 if cfg["d_model"] > 2048 else int(waves))
    g.sync()


def test_passes_of_both_kinds_take_turns():
    """Few messages take workgroups of four wavefronts, more of them workgroups of eight.  The two cut the residual products
    into different numbers of slices (here 8 and 16) and leave their partial results in the same arrays."""
    cfg = S.tiny(n_layer=2, dtype=S.DT_BF16, max_ctx=64, vocab=97, d_model=2048, n_head=8, n_kv_head=2, head_dim=64, d_ff=512)
    w = scale_matrices(S.make_weights(cfg, 47, exercise=True), 1.0)
    o, g = pair(cfg, w, 0, 2, embed=True, max_seqs=6, kv_page_tokens=8)
    for s, ids in enumerate(S.make_prompts(cfg, 47, 6, 7)):
        check(g.prefill(s, dev_ids(ids)), o.prefill(s, ids), cfg, ("prefill", s))
    rng = np.random.default_rng(3)
    for step, n in enumerate([4, 6, 2, 5, 3, 6, 4]):
        order = [int(s) for s in rng.permutation(6)[:n]]
        toks = [int(rng.integers(0, cfg["vocab"])) for _ in order]
        for s, t, got in zip(order, toks, g.decode_batch(order, [dev_ids([t]) for t in toks])):
            check(got, o.decode_step(s, t), cfg, ("batched decode", step, s))
        assert g.info(7) == (4 if n <= 4 else 8)
    g.sync()
