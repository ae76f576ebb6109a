"""The shared pass at a position whose angles lie 2^31 bytes into the table of them."""
import numpy as np
import pytest
import torch

from paper_2505_18164_amd import synth as S
from gpu_util import check, dev_ids, pair, scale_matrices

pytestmark = pytest.mark.gpu


def test_rotation_of_far_positions():
    """A sample of 2^22 positions (heads of 128: 512 bytes of angles each) and one of five take the same new token.  The
    query and key matrices are one and large, so the new position attends to itself (its score is above 50, the others
    together weigh less than e^27) and both samples have the oracle's result for the short one - if query and key are turned
    by the same angles, whatever these are; not turned at all, or not alike, attention would see the prompt's values."""
    far, piece = 1 << 22, 1 << 16
    cfg = S.tiny(n_layer=1, dtype=S.DT_BF16, max_ctx=far + 64, vocab=61, d_model=64, n_head=1, n_kv_head=1, head_dim=128, d_ff=64)
    w = scale_matrices(S.make_weights(cfg, 71, exercise=True), 2.0)
    qk = np.random.default_rng(71).standard_normal((128, 64)).astype(np.float32) * np.float32(0.3)
    w["layers"][0]["wq"] = w["layers"][0]["wk"] = S.storage_round(qk, cfg["dtype"])
    o, g = pair(cfg, w, 0, 1, embed=True, max_seqs=2, kv_page_tokens=64, kv_pages=far // 64 + 4, max_prefill=piece)
    ids = dev_ids(np.full(piece, 7))
    out = torch.empty((piece, cfg["d_model"]), dtype=torch.bfloat16, device="cuda:0")
    for _ in range(far // piece):
        g.prefill_chunk(0, ids, out)
    g.prefill(1, ids[:5])
    o.prefill(0, np.full(5, 7))
    for token in (11, 23):
        want = o.decode_step(0, token)
        for s, got in enumerate(g.decode_batch([0, 1], [dev_ids([token])] * 2)):
            check(got, want, cfg, ("decode", token, s))
    g.sync()
