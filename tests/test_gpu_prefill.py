"""GPU parity of prefills whose chunk is longer than the queries one attention workgroup holds (64 at head size 64, 32 at
head size 128) and of prefills of several chunks, at the edges of both."""
import numpy as np
import pytest

from paper_2511_13587_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gc():
    import gpu_common
    return gpu_common


@pytest.mark.parametrize("head,tokens,prompts", [(64, 64, 1), (64, 65, 2), (64, 127, 1), (64, 129, 1), (128, 33, 1), (128, 64, 2), (128, 97, 1),
                                                 (64, 513, 1), (64, 70, 33), (64, 320, 2), (64, 301, 3), (128, 97, 5), (128, 141, 5)])
def test_prefill_of_long_chunks_bf16(gc, head, tokens, prompts):
    """Last-position logits and the whole cache after `tokens` prefilled positions (513: a second chunk of one token; 33 prompts:
    a chunk of 64 tokens and one of 6; 2, 3 and 5 prompts: projections of one round of 128 x 128 tiles and of up to two)."""
    base = synth.B_SHAPE if head == 64 else synth.SEVEN_B.replace(d_model=1024, n_heads=8, d_ff=2752)
    # one layer: the cache of layer 0 depends on no attention, the logits do
    shape = base.replace(n_layers=1, n_prompts=prompts, n_nodes=2, tree_widths=None, vocab=1024, logit_lo=0, logit_hi=1024, grid_h=32, grid_w=32,
                         prefix_len=1, prefix_kind=synth.PREFIX_CLASS)
    sample = [0, prompts - 1] if prompts > 1 else [0]
    pair = gc.Pair(shape, gain_jitter=0.1, shadow=True, sample=sample)
    pair.prefill(n_forced=tokens - 1)
    raw, _, _ = pair.gpu_logits()
    d = raw[pair.rows(), 0] - pair.oracle.prefill_logits
    err = float(np.abs(d).max())
    print("prefill", head, tokens, "logit error", err, "floor", pair.floor)
    assert err <= gc.logit_tol(shape, pair.floor, pair.fused), (err, pair.floor)
    assert gc.rms(d) <= gc.logit_rms_tol(shape, pair.floor_rms, pair.fused)
    gc.check_kv(pair, 0, tokens, "prefill", prompts=sample)
    pair.close()
