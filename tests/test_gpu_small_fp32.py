"""GPU parity of the launch-bound fp32 layer (normalisation, rotary embedding, SwiGLU and residual sum inside the products) at the
edges of its tiles: contraction lengths around 64 and 128 pieces of 4, rows around the 8 of a wave, and both sides of the
limits beyond which the plain kernels run."""
import numpy as np
import pytest

from paper_2511_13587_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gc():
    import gpu_common
    return gpu_common


# (d, heads, d_ff, prompts, draft nodes, prefilled tokens): d and d_ff of 8, 256 and 264, 512 and 520 and 1024 values (2, 64, 66, 128, 130
# and 256 pieces); 8, 10, 16, 18 and 128 rows; 130 rows (plain kernels); a cache almost full
@pytest.mark.parametrize("d,heads,d_ff,prompts,nodes,tokens", [(8, 1, 8, 1, 3, 5), (256, 8, 264, 1, 4, 9), (264, 3, 256, 2, 3, 12), (512, 4, 520, 2, 7, 20),
                                                              (520, 5, 1024, 3, 2, 7), (1024, 8, 512, 1, 4, 33), (128, 4, 344, 1, 63, 31),
                                                              (128, 4, 344, 5, 12, 6), (128, 4, 344, 1, 5, 57)])
def test_small_layer_fp32(gc, d, heads, d_ff, prompts, nodes, tokens):
    shape = synth.TINY.replace(n_layers=2, d_model=d, n_heads=heads, d_ff=d_ff, n_prompts=prompts, n_nodes=nodes, grid_h=8 if nodes < 63 else 12,
                               grid_w=8 if nodes < 63 else 12, tree_widths=None)
    pair = gc.Pair(shape, gain_jitter=0.1)
    pair.prefill(n_forced=tokens)
    raw, _, _ = pair.gpu_logits()
    assert np.abs(raw[:, 0] - pair.oracle.prefill_logits).max() < 1e-4
    for call in range(2):
        parent = synth.tree_parents(None, nodes) if call else np.maximum(np.arange(nodes) - 2, 0).astype(np.int32)
        q, toks = synth.make_draft(shape, parent, call)
        pair.verify(parent, toks, q, synth.make_uniforms(shape, nodes, call))
        gc.check_logits(pair, f"d {d}, call {call}")
        for r in (0, 2 * prompts - 1):
            n = pair.oracle.kv_len(r // 2)
            k, v = pair.ctx.vvs_debug_kv(1, r, n)
            assert np.abs(k.cpu().numpy() - pair.oracle.kc[r][1][:n].reshape(n, -1)).max() < 1e-4
            assert np.abs(v.cpu().numpy() - pair.oracle.vc[r][1][:n].reshape(n, -1)).max() < 1e-4
        pair.commit()
    pair.close()


# d and d_ff of 264 values: 66 pieces of 4, so most lanes stand past the end of the second 64 and must add nothing, whatever the row's last piece
def test_infinities_in_the_last_piece(gc):
    shape = synth.TINY.replace(n_layers=1, d_model=264, n_heads=3, d_ff=264, tree_widths=None)
    w = synth.make_weights(shape)
    w["gf"][-1] = np.inf                       # final norm and head
    pair = gc.Pair(shape, weights=w)
    pair.prefill(n_forced=9, run_oracle=False)
    raw, _, _ = pair.gpu_logits()
    assert np.isinf(raw).all()                 # one infinite term beside finite ones
    sign = np.sign(raw[:, 0] * w["wout"][-1, shape.logit_lo:shape.logit_hi])
    assert (sign == sign[:, :1]).all()         # the sign of the row's last value, which every column shares
    pair.close()
    w = synth.make_weights(shape)
    w["l0.wg"][:, -1] *= 1e24                  # the last hidden unit leaves the range of fp32 where its gate is open
    w["l0.wu"][:, -1] *= 1e24
    pair = gc.Pair(shape, weights=w, feature_pre_norm=1)
    for n_forced in range(1, 8):
        pair.prefill(n_forced=n_forced)
        got = pair.ctx.vvs_read_features()[0][:, 0]
        want = np.stack([pair.oracle.features(r)[-1] for r in range(shape.n_rows)])
        far = np.abs(want) > 1e39
        assert np.array_equal(np.isposinf(got), far & (want > 0)) and np.array_equal(np.isneginf(got), far & (want < 0)), n_forced
        assert np.isfinite(got[~far]).all()
    pair.close()
