"""Wide layers (separate normalisations) of few rows in one launch: parity at the edges of its tiles, where it ends, and with repeated calls."""
import numpy as np
import pytest
import torch

from paper_2511_13587_amd import synth
from test_gpu_parity import gc, run_bf16_case, show  # noqa: F401
from test_gpu_shared_tiles import check_prefill

pytestmark = pytest.mark.gpu


# d 1536: 2 rows; 12 and 24 heads (head size 128, 64); 32, 34 and 64 rows, one row-block to a tile; 66, 98 and 128 rows, two; 130 rows, a launch per projection;
# d_ff no multiple of 48 and no whole share of 32 (4160 / 32 = 130); more pairs than CUs, so that rows share an attention unit.  d 2304: two from 34 rows on, up to 64
@pytest.mark.parametrize("d,heads,d_ff,prompts,tokens,n_forced", [
    (1536, 12, 4096, 1, 2, 9), (1536, 24, 4096, 1, 16, 40), (1536, 12, 4096, 1, 17, 70), (1536, 12, 4096, 1, 32, 33), (1536, 24, 4160, 2, 16, 31), (1536, 24, 4096, 8, 4, 20),
    (1536, 12, 4096, 16, 2, 20), (1536, 24, 4096, 3, 11, 20), (1536, 12, 4160, 7, 7, 20), (1536, 24, 4096, 4, 16, 20), (1536, 12, 4096, 13, 5, 9), (2304, 18, 2304, 1, 17, 20),
    (2304, 36, 2368, 2, 11, 20), (2304, 18, 2304, 4, 8, 20), (2304, 18, 2304, 3, 11, 20)])
def test_wide_layers_in_one_launch(gc, d, heads, d_ff, prompts, tokens, n_forced):  # noqa: F811
    shape = synth.SEVEN_B.replace(d_model=d, n_heads=heads, d_ff=d_ff, n_layers=2, vocab=1024, logit_lo=0, logit_hi=1024, prefix_len=8, n_prompts=prompts,
                                  n_nodes=tokens - 1, tree_widths=None)
    sample = {"sample": [0, prompts - 1]} if prompts > 4 else {}
    together = 2 * prompts * tokens <= (128 if d <= 2048 else 64)
    show(f"d {d} heads {heads} d_ff {d_ff} {prompts} x {tokens}", run_bf16_case(gc, shape, n_forced=n_forced, calls=2, one_launch=together, **sample))


# Prefills (positions from the prefill's base, one class token in front): 2, 28, 30 and 32 rows, one row-block to a tile, both head sizes; d_ff that gate/up
# as a launch of its own would split at d 4096 (SwiGLU by a division), and one of 16448 columns; a chunk of 512 tokens and one of 2 behind it
@pytest.mark.parametrize("d,heads,d_ff,tokens", [(1536, 12, 4096, 1), (2048, 16, 4096, 14), (4096, 32, 4096, 15), (1536, 24, 4160, 16), (2048, 16, 16448, 9), (1536, 12, 1536, 514)])
def test_prefill_of_wide_layers_in_one_launch(gc, d, heads, d_ff, tokens):  # noqa: F811
    check_prefill(gc, d, heads, d_ff, tokens, norm_mode=1 if d_ff == 1536 else 0, one_launch=tokens < 512 or None)


def test_gate_below_the_normal_range(gc):  # noqa: F811
    """SwiGLU with expf and a division, as the kernel for split gate/up sums has it: at a gate of -88 its sigmoid is 6e-39, below the normal range,
    which a reciprocal instruction gives as zero.  One hidden unit with an up value of 1e30 and a down weight of 2^20 makes it -0.7 of the residual stream."""
    shape = synth.SEVEN_B.replace(d_model=4096, n_heads=32, d_ff=1024, n_layers=1, vocab=1024, logit_lo=0, logit_hi=1024, prefix_len=1, n_prompts=1, n_nodes=0)
    rng = np.random.default_rng(3)
    w = {n: np.zeros(synth.weight_dims(shape, n), dtype=np.float32) for n in synth.weight_names(shape)}
    for n in w:
        if w[n].ndim == 1:
            w[n][:] = 1.0
    bf16 = lambda a: synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(np.asarray(a, dtype=np.float32)))   # noqa: E731
    w["embed"] = bf16(0.002 * rng.standard_normal(w["embed"].shape))
    w["embed"][:, 0] = 1.0                               # with the others 1.6 % of its square and 4096 eps: x / rms = 62.25
    w["l0.wg"][0, 5] = bf16(-88.0 / 62.25)[0]
    w["l0.wu"][0, 5] = 2.0 ** 94
    w["l0.wd"][5, 1:] = 2.0 ** 20
    pair = gc.Pair(shape, weights=w, with_oracle=False, feature_pre_norm=1)
    pair.prefill(n_forced=3, run_oracle=False)
    pending = int(pair.ctx.vvs_read_state()[2, 0])
    pair.ctx.vvs_timing_enable(True)
    pair.verify(None, None, None, synth.make_uniforms(shape, 0, 0), run_oracle=False)
    assert pair.ctx.vvs_timing_read(gc.vb.VVS_K_GEMM)[0] == 2                # the layers, the output head
    pair.ctx.vvs_timing_enable(False)
    pair.commit(run_oracle=False)
    features, count = pair.ctx.vvs_read_features()
    x = w["embed"][pending].astype(np.float64)
    h = bf16(x / np.sqrt(np.mean(x * x) + shape.rms_eps)).astype(np.float64)
    gate, up = h[0] * w["l0.wg"][0, 5], h[0] * np.float64(w["l0.wu"][0, 5])
    assert -88.7 < gate < -87.4
    x[1:] += bf16(gate / (1.0 + np.exp(-gate)) * up).astype(np.float64) * 2.0 ** 20
    # the exponential of a 32-bit argument of 88: 2^-18 of the value, which may move its bf16 rounding; and the feature's own rounding
    assert np.abs(features[:, count[0] - 1] - x).max() <= 2.0 ** -7 * np.abs(x[1:]).max()
    pair.close()
