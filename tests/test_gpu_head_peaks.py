"""Draws behind the shared vocabulary pass, which leaves the best logit of every wavefront's rows: vocabularies at the least
that takes this way, ragged ones, ones of several blocks per wavefront, and equal logits in more groups than are followed."""
import numpy as np
import pytest
import torch

from oracle import mdi_oracle as O
from paper_2505_18164_amd import mdi, synth as S
from gpu_util import dev_acts, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("equal_rows", [False, True])
@pytest.mark.parametrize("top_k", [2, 50, 64])
@pytest.mark.parametrize("vocab", [1025, 32769, 70001])
def test_draws_follow_the_oracle_sampler(vocab, top_k, equal_rows):
    cfg = S.tiny(n_layer=1, dtype=S.DT_BF16, max_ctx=32, vocab=vocab, d_model=64, n_head=4, n_kv_head=2, head_dim=16, d_ff=96)
    w = S.make_weights(cfg, 91, 1, 1, head=True, exercise=True)
    w["lm_head"] = S.storage_round(w["lm_head"] * np.float32(16.0), cfg["dtype"])
    if equal_rows:                                       # every row one of five: many groups share their best logit
        w["lm_head"] = np.ascontiguousarray(w["lm_head"][np.arange(vocab) % 5])
    g = mdi.Partition(cfg, w, 1, 1, has_head=True, max_seqs=8)
    n, seed, temperature = 5, 0x1234567890ABCDEF, 0.8
    xd = [dev_acts(S.make_activations(cfg, 92, s, 1)[0], cfg) for s in range(n)]
    lg = torch.empty((n, vocab), dtype=torch.float32, device="cuda:0")
    decided = 0
    for rnd in range(6):
        steps = [7 * rnd + i for i in range(n)]
        toks = host(g.sample_batch(list(range(n)), xd, temperature, top_k, seed, steps, logits_out=lg)).astype(np.int64)
        got = host(lg)
        for i in range(n):
            u = O.uniform01(seed, i, steps[i])
            pmf = O.topk_pmf(got[i].astype(np.float64), temperature, top_k)
            assert int(toks[i]) in pmf
            if np.abs(np.cumsum(list(pmf.values())) - u).min() > 1e-5:      # (binary32 sums of at most 64 weights)
                decided += 1
                assert int(toks[i]) == O.sample_topk(got[i], temperature, top_k, u), (rnd, i)
    assert decided >= 0.9 * 6 * n
    g.sync()
