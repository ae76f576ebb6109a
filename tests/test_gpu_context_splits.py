"""Where a sample's context begins to be split among workgroups, in the kernels for one message, for several and for a shared
pass, and the fold with one and with two query heads per work item."""
import numpy as np
import pytest

from paper_2505_18164_amd import synth as S
from gpu_util import check, dev_ids, pair, scale_matrices

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads", [1, 2], ids=["one head", "two heads"])
@pytest.mark.parametrize("norm", [S.NORM_LAYERNORM, S.NORM_RMSNORM], ids=["layernorm", "rmsnorm"])
@pytest.mark.parametrize("dtype", [S.DT_F32, S.DT_BF16], ids=["f32", "bf16"])
def test_samples_that_grow_across_the_limit(dtype, norm, heads, monkeypatch):
    monkeypatch.setenv("MDI_WHOLE_CTX", "260")
    monkeypatch.setenv("MDI_GROUP_CTX", "0" if heads == 2 else "4096")
    cfg = S.tiny(n_layer=2, dtype=dtype, max_ctx=512, vocab=97, d_model=64, n_head=4, n_kv_head=2, head_dim=16, d_ff=96, norm_kind=norm)
    w = scale_matrices(S.make_weights(cfg, 83, exercise=True), 3.0 if dtype == S.DT_F32 else 2.0)
    lens = (257, 9, 255)
    o, g = pair(cfg, w, 0, 2, embed=True, max_seqs=len(lens), kv_page_tokens=16)
    for s, T in enumerate(lens):
        ids = S.make_prompts(cfg, 83 + s, 1, T)[0]
        check(g.prefill(s, dev_ids(ids)), o.prefill(s, ids), cfg, ("prefill", s))
    rng = np.random.default_rng(2)
    calls = [("one", [0], 1), ("several", [2, 0, 1], 1), ("shared", [0, 2, 1], 1), ("one", [0], 3), ("several", [1, 0, 2], 3),
             ("shared", [2, 0, 1], 3), ("several", [1, 2], 1), ("shared", [1, 2], 3), ("one", [2], 3)]
    for step, (kind, order, splits) in enumerate(calls):
        toks = [int(rng.integers(0, cfg["vocab"])) for _ in order]
        ins = [dev_ids([t]) for t in toks]
        if kind == "one":
            outs = [g.decode_step(order[0], ins[0])]
        else:
            outs = (g.decode_steps if kind == "several" else g.decode_batch)(order, ins)
        for s, t, got in zip(order, toks, outs):
            check(got, o.decode_step(s, t), cfg, (kind, step, s))
        assert g.info(8) == splits, (step, [g.seq_len(s) for s in order])
    g.sync()


@pytest.mark.parametrize("dtype", [S.DT_F32, S.DT_BF16], ids=["f32", "bf16"])
def test_default_limit(dtype):
    """64 KiB of one head's keys and values with workgroups of four wavefronts (several messages), 96 KiB with eight (one):
    heads of 16 need 64 bytes a position in bf16, twice that in fp32."""
    four = 64 * 1024 // (64 if dtype == S.DT_BF16 else 128)
    cfg = S.tiny(n_layer=2, dtype=dtype, max_ctx=2048, vocab=97, d_model=64, n_head=4, n_kv_head=2, head_dim=16, d_ff=96)
    w = scale_matrices(S.make_weights(cfg, 89, exercise=True), 2.0)
    lens = (four - 1, 9, four * 3 // 2 - 1)
    o, g = pair(cfg, w, 0, 2, embed=True, max_seqs=len(lens), kv_page_tokens=16)
    for s, T in enumerate(lens):
        ids = S.make_prompts(cfg, 89 + s, 1, T)[0]
        check(g.prefill(s, dev_ids(ids)), o.prefill(s, ids), cfg, ("prefill", s))
    for step, (order, waves, splits) in enumerate([([0, 1], 4, 1), ([0], 8, 1), ([1, 0], 4, four // 128 + 1), ([2], 8, 1),
                                                   ([2], 8, four * 3 // 256 + 1)]):
        ins = [dev_ids([t + step]) for t in order]
        outs = [g.decode_step(order[0], ins[0])] if len(order) == 1 else g.decode_batch(order, ins)
        for s, got in zip(order, outs):
            check(got, o.decode_step(s, s + step), cfg, (step, s))
        assert (g.info(7), g.info(8)) == (waves, splits), step
    g.sync()
