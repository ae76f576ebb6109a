"""mdi_partition_trace records the moments include/mdi.h names, in their order."""
import numpy as np
import pytest
import torch

from paper_2505_18164_amd import mdi, synth as S
from gpu_util import dev_acts, host

pytestmark = pytest.mark.gpu

QKV, ATTN, OPROJ, UP, DOWN = range(5)


def traced(n, shared):
    cfg = S.tiny(n_layer=3, dtype=S.DT_BF16, max_ctx=512, vocab=61, d_model=2048, n_head=32, n_kv_head=8, head_dim=64, d_ff=4096)
    g = mdi.Partition(cfg, S.make_weights(cfg, 80), 0, 3, max_seqs=n)
    for s in range(n):
        g.prefill(s, dev_acts(S.make_activations(cfg, 81, s, 40), cfg))
    xs = [dev_acts(S.make_activations(cfg, 82, s, 1)[0], cfg) for s in range(n)]
    buf = torch.zeros((2, g.info(1), 3, 5, 8), dtype=torch.int64, device="cuda:0")
    step = (lambda: g.decode_batch(list(range(n)), xs)) if shared else (lambda: g.decode_steps(list(range(n)), xs))
    step()                                               # a first launch waits for its code
    g.trace(buf)
    step()
    g.sync()
    g.trace(None)
    return buf.cpu().numpy()


def in_order(t, slots):
    """t [workgroups, layers, 8]: the slots are all set and do not go back."""
    v = t[..., slots]
    assert (v > 0).all()
    assert (np.diff(v, axis=-1) >= 0).all()


@pytest.mark.parametrize("n", [1, 4])
def test_one_pass_per_message(n):
    """Entering a phase, asking for its vector and issuing two tiles takes a microsecond (100 ticks): the first two
    slots are apart."""
    for t in traced(n, False)[:1 if n == 1 else 2]:
        for ph in (QKV, OPROJ, UP, DOWN):
            in_order(t[:, :, ph], [0, 1, 2, 3, 4, 5, 6])
            assert np.median(t[:, :, ph, 1] - t[:, :, ph, 0]) >= 10, ph
            assert (t[:, :, ph, 7] == 0).all()
        in_order(t[:, :, ATTN], [0, 1, 2, 3, 5, 6])
        assert np.median(t[:, :, ATTN, 1] - t[:, :, ATTN, 0]) >= 10


def test_one_pass_for_all_messages():
    t = traced(4, True)[0]
    for ph in (QKV, UP):
        in_order(t[:, :, ph], [0, 1, 2, 3, 4, 5, 6])
        assert (t[:, :, ph, 7] == 0).all()
    for ph in (OPROJ, DOWN):
        in_order(t[:, :, ph], [0, 1, 2, 3, 7, 5, 6])
        assert (t[:, :, ph, 4] == 0).all()
    items = t[:, 0, ATTN, 1] > 0                         # 128 work items of 40 positions for 256 workgroups
    assert items.sum() >= 32
    in_order(t[items][:, :, ATTN], [0, 1, 2, 3, 5, 6])
