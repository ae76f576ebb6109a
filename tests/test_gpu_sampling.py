"""The draw from the top-k tempered pmf at the sizes where the selection of the candidates changes: vocabularies that
are candidates as a whole, rows that start off a 16-byte boundary, and logits that tie en masse (more of them reach
the bound than the kernel keeps, so the ranks are found one after the other)."""
import numpy as np
import pytest
import torch

from oracle import mdi_oracle as O
from paper_2505_18164_amd import mdi, synth as S
from gpu_util import dev_acts, host

pytestmark = pytest.mark.gpu


def head(vocab, seed, lm_head=None, d=64):
    cfg = S.tiny(n_layer=1, d_model=d, n_head=4, n_kv_head=4, head_dim=16, d_ff=2 * d, vocab=vocab, dtype=S.DT_BF16)
    w = S.make_weights(cfg, seed, 1, 1, embed=False, head=True, exercise=True)
    w["lm_head"] = w["lm_head"] * np.float32(10.0) if lm_head is None else lm_head(w["lm_head"])
    return cfg, mdi.Partition(cfg, w, 1, 1, has_head=True, max_seqs=8)


def check_draws(cfg, g, top_k, n, seed=0x1234_5678_9ABC_DEF0, temperature=0.9, rounds=6):
    xs = [dev_acts(S.make_activations(cfg, 5, s, 1)[0], cfg) for s in range(n)]
    lg = torch.empty((n, cfg["vocab"]), dtype=torch.float32, device="cuda:0")
    decided = 0
    for step in range(rounds):
        toks = host(g.sample_batch(list(range(n)), xs, temperature, top_k, seed, [step] * n, logits_out=lg)).astype(np.int64)
        got = host(lg)
        for i in range(n):
            u = O.uniform01(seed, i, step)
            pmf = O.topk_pmf(got[i].astype(np.float64), temperature, top_k)
            assert int(toks[i]) in pmf, (i, step)
            if np.abs(np.cumsum(list(pmf.values())) - u).min() > 1e-5:   # binary32 sums of up to 64 weights: 64 * 2^-24
                decided += 1
                assert int(toks[i]) == O.sample_topk(got[i], temperature, top_k, u), (i, step)
    assert decided >= 0.9 * rounds * n
    g.sync()


# 1024 / 1025: everything is a candidate / the bound is looked for; odd widths: rows 1, 2 and 3 start at every offset
# inside a 16-byte piece; 33000: several rounds of pieces per thread
@pytest.mark.parametrize("vocab,top_k", [(64, 64), (97, 5), (1024, 64), (1025, 64), (1027, 1), (4099, 50), (33001, 64), (33001, 2)])
def test_draws_follow_the_oracle_sampler(vocab, top_k):
    cfg, g = head(vocab, 3)
    check_draws(cfg, g, top_k, n=5)
    check_draws(cfg, g, top_k, n=1)


# rows of the vocabulary matrix that repeat give logits that are equal to the last bit: 3000 of one value, and 40 values
# 100 times each (so that ties straddle the k-th rank)
@pytest.mark.parametrize("distinct", [1, 40])
def test_masses_of_equal_logits(distinct):
    cfg, g = head(3000 if distinct == 1 else 4000, 4, lambda m: np.tile(m[:distinct] * np.float32(10.0), (m.shape[0] // distinct, 1)))
    check_draws(cfg, g, 20, n=3)
    check_draws(cfg, g, 64, n=1)


# what the logits are beside a few ordinary ones, how many are ordinary, vocabulary, k: a few NaNs among the candidates
# (both sides of the size from which the bound is looked for); fewer than k numbers, which leaves the ranks to the rounds
# (also where threads own no element); -inf en masse, where the bound is -inf and everything reaches it; -inf that is
# ranked but never drawn
@pytest.mark.parametrize("rest,ordinary,vocab,top_k", [("nan", 90, 97, 20), ("nan", 1000, 1024, 64), ("nan", 4000, 4099, 50),
                                                       ("nan", 14, 97, 64), ("nan", 10, 1025, 50), ("nan", 3, 33001, 64),
                                                       ("-inf", 10, 1000, 50), ("-inf", 10, 1025, 50), ("-inf", 10, 33001, 64),
                                                       ("-inf", 3000, 4099, 64)])
def test_logits_that_are_no_ordinary_numbers(rest, ordinary, vocab, top_k):
    rows = np.random.default_rng(vocab).permutation(vocab)[ordinary:]

    def mat(m):
        m = m * np.float32(10.0)
        m[rows] = 0.0
        m[rows, 0] = np.nan if rest == "nan" else -np.inf            # times a positive activation
        return m

    cfg, g = head(vocab, 6, mat)
    n, seed, temperature = 3, 77, 0.9
    acts = [S.make_activations(cfg, 8, s, 1)[0] for s in range(n)]
    for a in acts:
        a[0] = 2.0
    xs = [dev_acts(a, cfg) for a in acts]
    lg = torch.empty((n, vocab), dtype=torch.float32, device="cuda:0")
    decided, rounds = 0, 6
    for count in (n, 1):                                             # the shared vocabulary pass and the one-sample kernel
        for step in range(rounds):
            toks = host(g.sample_batch(list(range(count)), xs[:count], temperature, top_k, seed, [step] * count, logits_out=lg)).astype(np.int64)
            got = host(lg)
            for i in range(count):
                assert np.isfinite(got[i]).sum() == ordinary
                assert not np.isposinf(got[i]).any()
                numbers = np.where(np.isnan(got[i]), np.float32(-np.inf), got[i])
                u = O.uniform01(seed, i, step)
                pmf = O.topk_pmf(numbers.astype(np.float64), temperature, top_k)
                assert pmf.get(int(toks[i]), 0.0) > 0.0, (i, step)
                if np.abs(np.cumsum(list(pmf.values())) - u).min() > 1e-5:
                    decided += 1
                    assert int(toks[i]) == O.sample_topk(numbers, temperature, top_k, u), (i, step)
    assert decided >= 0.9 * rounds * (n + 1)
    g.sync()
