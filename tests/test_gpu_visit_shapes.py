"""First visits at the numbers of positions and widths where the products' tiles change: one position, one more and one
less than a tile, inner dimensions that end inside a 128-byte step (520 and 4104 values), and enough positions for the
larger tiles; the numbers of positions also move how the inner dimension is split.  Against the oracle, every position
on its own, at the bar of the storage type."""
import numpy as np
import pytest
import torch

from paper_2505_18164_amd import mdi, synth as S
import visit_cases as V
from gpu_util import check, dev_acts, host, pair

pytestmark = pytest.mark.gpu


def ragged(**kw):
    base = dict(n_layer=1, d_model=520, n_head=8, n_kv_head=4, head_dim=64, d_ff=4104, vocab=61, max_ctx=2304, dtype=S.DT_BF16)
    base.update(kw)
    return S.tiny(**base)


F32 = dict(dtype=S.DT_F32)
GELU = dict(norm_kind=S.NORM_LAYERNORM, mlp_kind=S.MLP_GELU_TANH, has_bias=1)


@pytest.mark.parametrize("T,kw", [(T, {}) for T in (1, 31, 32, 33, 64, 65, 130, 257, 700, 2050)] + [(T, GELU) for T in (16, 129, 515)]
                         + [(T, F32) for T in (1, 32, 33, 64, 65, 200, 700)] + [(T, dict(GELU, **F32)) for T in (31, 300)],
                         ids=lambda v: v if isinstance(v, int) else ("f32_" if "dtype" in v else "bf16_") + ("gelu" if "mlp_kind" in v else "swiglu"))
def test_first_visits_across_tile_edges(T, kw):
    cfg = ragged(**kw)
    w = S.make_weights(cfg, 50, exercise=True)
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
    x = S.make_activations(cfg, 51, 0, T)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", T))
    y = S.make_activations(cfg, 52, 0, 1)[0]
    check(g.decode_step(0, dev_acts(y, cfg)), o.decode_step(0, y), cfg, ("later visit after", T))
    g.sync()


# ... and the sizes at which the choice of tiles falls on the (product, tile shape) pairs that neither these nor the
# benchmark shapes reach: every shape in every epilogue it can have, none of the sizes a multiple of its tiles
@pytest.mark.parametrize("dtype,d,heads,kv,h,d_ff,T", [
    (S.DT_BF16, 72, 2, 2, 64, 24, 9), (S.DT_BF16, 3080, 2, 2, 64, 520, 1300), (S.DT_BF16, 1032, 2, 2, 64, 6152, 1300),
    (S.DT_BF16, 72, 32, 8, 64, 2056, 2050), (S.DT_BF16, 3080, 2, 2, 64, 2056, 3000), (S.DT_BF16, 72, 2, 2, 64, 6152, 2050),
    (S.DT_BF16, 3080, 64, 32, 128, 24, 700), (S.DT_BF16, 6152, 2, 2, 64, 24, 2050),
    (S.DT_F32, 520, 24, 8, 64, 72, 300), (S.DT_F32, 3080, 2, 2, 64, 72, 257), (S.DT_F32, 2056, 2, 2, 64, 1032, 700), (S.DT_F32, 2056, 2, 2, 64, 520, 700)])
def test_first_visits_with_every_tile_shape(dtype, d, heads, kv, h, d_ff, T):
    mlp = {} if (dtype, d_ff) == (S.DT_F32, 520) else GELU           # (gate and up, the others: one matrix and biases)
    cfg = S.tiny(n_layer=1, d_model=d, n_head=heads, n_kv_head=kv, head_dim=h, d_ff=d_ff, vocab=61, max_ctx=T, **{**mlp, "dtype": dtype})
    w = S.make_weights(cfg, 55, exercise=True)
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
    x = S.make_activations(cfg, 56, 0, T)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", T))
    g.sync()


# Tiles of 256 x 256, 256 x 192, 192 x 192, 128 x 192, 96 x 128 and 64 x 96: each in the QKV, split, residual and MLP product
@pytest.mark.parametrize("T,d,heads,kv,d_ff,mlp", [
    (2090, 72, 32, 32, 2056, GELU), (1473, 72, 2, 2, 4104, {}),                                                    # 256 x 256
    (1068, 72, 32, 32, 2056, GELU), (973, 3080, 8, 2, 5512, GELU), (1971, 3080, 2, 1, 24, GELU), (1199, 72, 2, 2, 5144, GELU),   # 256 x 192
    (1408, 1032, 32, 32, 24, GELU), (1182, 3208, 4, 1, 4104, {}), (2475, 3080, 16, 2, 24, {}), (688, 1032, 4, 4, 5656, {}),      # 192 x 192
    (543, 72, 32, 32, 5360, GELU), (328, 3080, 64, 2, 24, GELU), (1195, 3080, 2, 1, 24, GELU), (394, 72, 2, 2, 4104, {}),        # 128 x 192
    (400, 72, 32, 32, 24, GELU), (2092, 1032, 2, 1, 4104, GELU), (195, 72, 2, 1, 4104, {}),                        # 96 x 128
    (70, 72, 16, 4, 24, GELU), (267, 1032, 2, 2, 24, GELU), (83, 72, 4, 2, 2056, {})])                             # 64 x 96
def test_first_visits_with_tiles_that_are_no_power_of_two(T, d, heads, kv, d_ff, mlp):
    cfg = S.tiny(n_layer=1, d_model=d, n_head=heads, n_kv_head=kv, head_dim=64, d_ff=d_ff, vocab=61, max_ctx=T, **{**mlp, "dtype": S.DT_BF16})
    w = S.make_weights(cfg, 57, exercise=True)
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
    x = S.make_activations(cfg, 58, 0, T)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", T))
    g.sync()


# The QKV product rotates and scatters from its tiles: heads of every size, longer than a tile and shorter, tiles of 192, 96 and
# 64 rows that begin inside a head of 128 or 256, positions rotated or not; a second piece that begins inside a page.
@pytest.mark.parametrize("T,d,h,heads,kv,kw", [
    (1408, 1032, 256, 8, 8, {}), (1408, 1032, 128, 16, 16, GELU), (400, 72, 256, 8, 8, {}), (400, 72, 128, 16, 16, {}),
    (333, 520, 128, 9, 3, {}), (37, 72, 256, 3, 1, GELU), (333, 72, 8, 6, 3, {}), (65, 520, 16, 12, 2, dict(GELU, pos_kind=S.POS_LEARNED)),
    (130, 72, 32, 5, 5, dict(pos_kind=S.POS_LEARNED)), (65, 72, 256, 3, 3, F32), (100, 520, 64, 10, 2, F32), (33, 72, 8, 4, 2, dict(GELU, **F32))])
def test_rotation_and_scatter_of_every_head_size(T, d, h, heads, kv, kw):
    cfg = S.tiny(n_layer=1, d_model=d, n_head=heads, n_kv_head=kv, head_dim=h, d_ff=72, vocab=61, max_ctx=T + 21, **{"dtype": S.DT_BF16, **kw})
    w = S.make_weights(cfg, 64, exercise=True)
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
    x = S.make_activations(cfg, 65, 0, T + 20)
    want = o.prefill(0, x)
    check(g.prefill(0, dev_acts(x[:T], cfg)), want[:T], cfg, ("first piece", T))
    check(g.prefill_chunk(0, dev_acts(x[T:], cfg)), want[T:], cfg, ("second piece after", T))
    y = S.make_activations(cfg, 66, 0, 1)[0]
    check(g.decode_step(0, dev_acts(y, cfg)), o.decode_step(0, y), cfg, ("later visit after", T))
    g.sync()


@pytest.mark.parametrize("T", [5, 300])
def test_output_rows_off_a_16_byte_boundary(T):
    cfg = ragged()
    w = S.make_weights(cfg, 60, exercise=True)
    g = mdi.Partition(cfg, w, 0, 1, max_seqs=2)
    x = dev_acts(S.make_activations(cfg, 61, 0, T), cfg)
    buf = torch.full((T * 520 + 2,), 7.0, dtype=torch.bfloat16, device="cuda:0")
    g.prefill(0, x, buf[1:T * 520 + 1].view(T, 520))
    want = g.prefill(1, x)
    g.sync()
    got = host(buf)
    assert got[0] == 7.0 and got[-1] == 7.0
    assert np.array_equal(got[1:-1].reshape(T, 520), host(want))


@pytest.mark.parametrize("kw", [{}, F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("d,T", [(520, 5), (8200, 3)])
def test_input_rows_off_a_boundary_of_four_values(d, T, kw):
    """(Rows of 8200 values are not held in registers.)"""
    cfg = ragged(d_model=d, d_ff=72, **kw)
    g = mdi.Partition(cfg, S.make_weights(cfg, 62, exercise=True), 0, 1, max_seqs=2)
    x = dev_acts(S.make_activations(cfg, 63, 0, T), cfg)
    buf = torch.zeros((T * d + 2,), dtype=x.dtype, device="cuda:0")
    off = buf[1:T * d + 1].view(T, d)
    off.copy_(x)
    got, want = g.prefill(0, off), g.prefill(1, x)
    g.sync()
    assert np.array_equal(host(got), host(want))


@pytest.mark.parametrize("page,heads,kv,h,cuts", [(64, 4, 2, 128, (130, 62, 1, 200)), (128, 4, 4, 64, (1, 127, 129, 64)), (48, 4, 1, 128, (100, 93, 7)),
                                                  (16, 4, 2, 64, (15, 17, 96, 200)), (5, 2, 2, 64, (64, 70)), (64, 32, 8, 64, (1600,)),
                                                  (24, 32, 4, 128, (1540, 3)),
                                                  # around the rule between 64 and 128 queries per workgroup (128 items of 128 queries)
                                                  (64, 16, 4, 128, (1024, 65, 1)), (64, 16, 4, 128, (1025, 63)), (24, 16, 8, 64, (1089, 95)), (64, 8, 8, 128, (1, 31, 33, 64, 66)),
                                                  # ... and between two and four groups (320 keys on average)
                                                  (64, 8, 2, 128, (639, 1, 64, 65)), (16, 8, 8, 64, (319, 2, 1, 200)), (64, 8, 8, 128, (640,)), (128, 8, 4, 64, (700, 33))])
def test_first_visits_read_keys_and_values_from_the_pages(page, heads, kv, h, cuts):
    """Pages that hold a block of 64 keys and pages that do not, both head sizes, pieces that end inside pages and blocks,
    and enough query blocks for workgroups of one group of wavefronts (384 of them); every position on its own."""
    cfg = S.tiny(n_layer=1, d_model=64, n_head=heads, n_kv_head=kv, head_dim=h, d_ff=96, vocab=61, max_ctx=1664, dtype=S.DT_BF16)
    w = S.make_weights(cfg, 70, exercise=True)
    o, g = pair(cfg, w, 0, 1, max_prefill=max(cuts), kv_page_tokens=page, max_seqs=2)
    g.prefill(1, dev_acts(S.make_activations(cfg, 72, 1, 33), cfg))     # the sample's pages do not begin the pool
    T = sum(cuts)
    x = S.make_activations(cfg, 71, 0, T)
    want = o.prefill(0, x)
    at = 0
    for n in cuts:
        check(g.prefill_chunk(0, dev_acts(x[at:at + n], cfg)), want[at:at + n], cfg, ("piece at", at))
        at += n
    y = S.make_activations(cfg, 73, 0, 1)[0]
    check(g.decode_step(0, dev_acts(y, cfg)), o.decode_step(0, y), cfg, ("later visit after", T))
    g.sync()


# Each launch of the attention: one group of wavefronts, two of four, two of two, four
@pytest.mark.parametrize("far", V.FAR)
@pytest.mark.parametrize("heads,kv,h,T", V.FAR_VISITS)
def test_scores_far_above_those_of_the_first_keys(heads, kv, h, T, far):
    """The first 256 keys, which every group begins with, lie 2^26 or 2^120 powers of two below the later ones: what is
    left of them does not touch the later scores."""
    cfg, w, x = V.far_visit(heads, kv, h, T, far)
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", T, V.launch_of(T, 0, heads)))
    g.sync()


@pytest.mark.parametrize("kw", [{}, GELU, F32], ids=["bf16_rms", "bf16_ln", "f32_rms"])
@pytest.mark.parametrize("d", [1016, 1032, 2056, 4104, 8184, 8200])
def test_norms_across_row_widths(d, kw):
    """A row is held in 1, 2, 4 or 8 pieces per thread, beyond 8192 values in none; few positions, so that the products
    before the norms leave partial results to add (their inner dimension, 2048, is split)."""
    cfg = S.tiny(n_layer=2, d_model=d, n_head=32, n_kv_head=2, head_dim=64, d_ff=2048, vocab=61, max_ctx=16, **{"dtype": S.DT_BF16, **kw})
    w = S.make_weights(cfg, 90, exercise=True)
    o, g = pair(cfg, w, 0, 2)
    x = S.make_activations(cfg, 91, 0, 5)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", d))
    g.sync()


@pytest.mark.parametrize("kw", [{}, GELU, F32], ids=["bf16_rms", "bf16_ln", "f32_rms"])
@pytest.mark.parametrize("d", [1016, 1032, 2056, 4104, 8184, 8200])
def test_norms_of_rows_without_partial_results(d, kw):
    """Inner dimensions of one step (32 values), which are not split."""
    cfg = S.tiny(n_layer=2, d_model=d, n_head=1, n_kv_head=1, head_dim=32, d_ff=32, vocab=61, max_ctx=16, **{"dtype": S.DT_BF16, **kw})
    w = V.loud(cfg, S.make_weights(cfg, 92, exercise=True))
    o, g = pair(cfg, w, 0, 2)
    x = S.make_activations(cfg, 93, 0, 5)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", d))
    g.sync()
