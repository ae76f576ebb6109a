"""First visits at the numbers of positions and widths where the products' tiles change: one position, one more and one
less than a tile, inner dimensions that end inside a 128-byte step (520 and 4104 values), and enough positions for the
larger tiles; the numbers of positions also move how the inner dimension is split.  Against the oracle, every position
on its own, at the bar of the storage type.  The inputs (visit_cases.py) are such that every product and the attention move
the rows by more than the bar, which test_visit_cases.py asserts."""
import numpy as np
import pytest
import torch

from paper_2505_18164_amd import mdi, synth as S
import visit_cases as V
from gpu_util import check, dev_acts, host, pair

pytestmark = pytest.mark.gpu


GELU, F32, ragged = V.GELU, V.F32, V.ragged


@pytest.mark.parametrize("T,kw", V.EDGES, ids=lambda v: v if isinstance(v, int) else ("f32_" if "dtype" in v else "bf16_") + ("gelu" if "mlp_kind" in v else "swiglu"))
def test_first_visits_across_tile_edges(T, kw):
    cfg = ragged(**kw)
    w = V.loud(cfg, S.make_weights(cfg, 50, exercise=True))
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
    x = S.make_activations(cfg, 51, 0, T)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", T))
    y = S.make_activations(cfg, 52, 0, 1)[0]
    check(g.decode_step(0, dev_acts(y, cfg)), o.decode_step(0, y), cfg, ("later visit after", T))
    g.sync()


# ... and the sizes at which the choice of tiles falls on the (product, tile shape) pairs that these do not reach
@pytest.mark.parametrize("dtype,T,d,heads,kv,h,d_ff,mlp", V.TILES)
def test_first_visits_with_every_tile_shape(dtype, T, d, heads, kv, h, d_ff, mlp):
    cfg, w, x = V.tile_visit(dtype, T, d, heads, kv, h, d_ff, mlp)
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
    check(g.prefill(0, dev_acts(x, cfg)), o.prefill(0, x), cfg, ("first visit", T))
    g.sync()


# The QKV product rotates and scatters from its tiles: heads of every size, longer than a tile and shorter, tiles of 192, 96 and
# 64 rows that begin inside a head of 128 or 256, positions rotated or not; a second piece that begins inside a page.
@pytest.mark.parametrize("T,d,h,heads,kv,kw", V.HEADS)
def test_rotation_and_scatter_of_every_head_size(T, d, h, heads, kv, kw):
    cfg, w, x = V.heads_visit(T, d, h, heads, kv, kw)
    o, g = pair(cfg, w, 0, 1, max_prefill=T)
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


@pytest.mark.parametrize("levels", V.LEVELS)
@pytest.mark.parametrize("page,heads,kv,h,cuts", V.PAGES)
def test_first_visits_read_keys_and_values_from_the_pages(page, heads, kv, h, cuts, levels):
    """Pages that hold a block of 64 keys and pages that do not, both head sizes, pieces that end inside pages and blocks,
    and every launch of the attention; scores that raise their references again and again, in some queries of a wavefront and
    not in others, and groups of wavefronts whose references are far apart; every position on its own."""
    cfg, w, x = V.pages_visit(heads, kv, h, cuts, levels)
    o, g = pair(cfg, w, 0, 1, max_prefill=max(cuts), kv_page_tokens=page, max_seqs=2)
    g.prefill(1, dev_acts(S.make_activations(cfg, 72, 1, 33), cfg))     # the sample's pages do not begin the pool
    T = sum(cuts)
    want = o.prefill(0, x[:T])
    at = 0
    for n in cuts:
        check(g.prefill_chunk(0, dev_acts(x[at:at + n], cfg)), want[at:at + n], cfg, ("piece at", at, V.launch_of(n, at, heads)))
        at += n
    check(g.decode_step(0, dev_acts(x[T], cfg)), o.decode_step(0, x[T]), cfg, ("later visit after", T))
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


def test_weights_are_summed_as_they_are_multiplied():
    """A weight is rounded to bf16 for the product with the values.  Where a few keys have all of it, the sum has to be of the
    rounded ones, or the output is off by another 2^-9: 2.61e-3 from the oracle over all rows, 2.71e-3 with a sum of the
    others, 2.60e-3 when the largest weight is always 1.  (The oracle rounds nothing; the bar is half way.)"""
    cfg, w, x = V.dominated_visit()
    o, g = pair(cfg, w, 0, 1, max_prefill=len(x))
    want = o.prefill(0, x)
    got = g.prefill(0, dev_acts(x, cfg))
    assert np.linalg.norm(host(got) - want) / np.linalg.norm(want) < 2.66e-3
    check(got, want, cfg, "first visit")
    g.sync()


@pytest.mark.parametrize("kw", [{}, GELU, F32], ids=["bf16_rms", "bf16_ln", "f32_rms"])
@pytest.mark.parametrize("d", [1016, 1032, 2056, 4104, 8184, 8200])
def test_norms_across_row_widths(d, kw):
    """A row is held in 1, 2, 4 or 8 pieces per thread, beyond 8192 values in none; few positions, so that the products
    before the norms leave partial results to add (their inner dimension, 2048, is split)."""
    cfg = S.tiny(n_layer=2, d_model=d, n_head=32, n_kv_head=2, head_dim=64, d_ff=2048, vocab=61, max_ctx=16, **{"dtype": S.DT_BF16, **kw})
    w = V.loud(cfg, S.make_weights(cfg, 90, exercise=True))
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
