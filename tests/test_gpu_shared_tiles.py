"""GPU parity of the projections that share their operands through LDS, at the edges of the tiles that large weights take:
plain products with and without a split of the contraction, and the q/k/v and gate/up epilogues."""
import numpy as np
import pytest

from paper_2511_13587_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gc():
    import gpu_common
    return gpu_common


def bf16_round(a):
    return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(np.asarray(a, dtype=np.float32)))


# rows, columns, contraction; the tile and the shares of the contraction that the planner takes (test_host_sanitized.py checks these on the CPU, so
# that a case cannot drift off its tile).  One row into the next tile, and 130 stages of the contraction in 4 shares (the last one is shorter).
PRODUCTS = [(33, 4096, 4096, (64, 64, 4)), (64, 4096, 4160, (64, 64, 4)), (65, 4096, 4096, (128, 64, 4)), (128, 4096, 4160, (128, 64, 4)),
            (129, 4096, 4096, (192, 64, 4)), (192, 4096, 11008, (192, 64, 4)), (193, 4096, 4096, (128, 64, 2)), (257, 4096, 4160, (192, 64, 2)),
            (388, 4096, 11008, (128, 128, 2)), (513, 4096, 4096, (192, 128, 2)), (130, 1536, 8192, (64, 128, 7)), (769, 4096, 11008, (256, 128, 2)),
            (1025, 4096, 11008, (256, 256, 3)), (1537, 4096, 11008, (256, 256, 2)), (1025, 4096, 4096, (192, 128, 1)), (2457, 2560, 512, (128, 128, 1))]


@pytest.mark.parametrize("m,n,k", [case[:3] for case in PRODUCTS])
def test_product_of_large_weights_bf16(gc, m, n, k):
    pair = gc.Pair(synth.B_SHAPE.replace(n_layers=1, n_prompts=1, vocab=1024, logit_hi=1024), with_oracle=False)
    rng = np.random.default_rng(m + n + k)
    a = bf16_round(rng.standard_normal((m, k)))
    w = bf16_round(rng.standard_normal((k, n)) * 0.05)
    got = pair.ctx.vvs_debug_gemm(gc.vb.to_device(a, 1), gc.vb.to_device(w, 1), m, n, k).cpu().numpy()
    want = a.astype(np.float64) @ w.astype(np.float64)
    # fp32 sums of k exact products of size 0.05: rounding noise of about sqrt(k) * 2^-24 times the sums' size sqrt(k) * 0.05
    scale = np.sqrt(k) * 0.05
    assert np.abs(got - want).max() < 2e-5 * scale * 10, np.abs(got - want).max()
    pair.close()


# d_model, heads, d_ff, tokens (rows = 2 x tokens); the tiles of q/k/v and of gate/up, both with whole sums (checked on the CPU as above; gate/up on
# 64 columns has operands of its own)
EPILOGUES = [(2048, 32, 3072, 24, (64, 64), (64, 64)), (2048, 16, 3072, 65, (128, 64), (64, 128)), (2048, 16, 3072, 150, (64, 128), (64, 128)),
             (2048, 32, 3072, 200, (128, 128), (128, 128)), (2048, 32, 3072, 345, (192, 128), (192, 128)), (2048, 16, 3072, 497, (128, 128), (256, 128)),
             (4096, 32, 1536, 90, (192, 64), (64, 64)), (4096, 32, 1536, 193, (256, 128), (64, 128)), (4096, 64, 1536, 194, (256, 128), (64, 128))]


@pytest.mark.parametrize("d,heads,d_ff,tokens", [case[:4] for case in EPILOGUES])
def test_epilogues_of_large_weights_bf16(gc, d, heads, d_ff, tokens):
    check_prefill(gc, d, heads, d_ff, tokens)


# d_model, heads, d_ff, tokens; tile and shares of gate/up where it keeps operands of its own (checked on the CPU as above): one round of CUs with whole sums,
# with sums in two shares, one row into the next row-block, and three rounds.  Up to 32 rows beyond d 4096, where not all layers are one launch
OWN_GATE_UP = [(4160, 65, 4160, 14, (32, 64, 1)), (2048, 32, 4096, 33, (64, 64, 1)), (4160, 65, 4096, 15, (32, 64, 2)), (4096, 32, 4096, 17, (64, 64, 2)),
               (4160, 65, 16448, 9, (32, 64, 1))]


@pytest.mark.parametrize("d,heads,d_ff,tokens", [case[:4] for case in OWN_GATE_UP])
def test_gate_up_with_operands_of_its_own_bf16(gc, d, heads, d_ff, tokens):
    check_prefill(gc, d, heads, d_ff, tokens)


# Projections of one shape: d_ff of 2 d has the down projection's contraction in common with a drafter's input map, d_ff of d / 2 the columns of
# gate/up with O's.  These row counts take more partial sums than the widest call.
@pytest.mark.parametrize("d,heads,d_ff,tokens,norm_mode", [(2560, 20, 5120, 464, 0), (3584, 28, 1792, 288, 0), (512, 8, 1024, 512, 1)])
def test_partial_sums_of_projections_alike_bf16(gc, d, heads, d_ff, tokens, norm_mode):
    check_prefill(gc, d, heads, d_ff, tokens, norm_mode)


def check_prefill(gc, d, heads, d_ff, tokens, norm_mode=0, one_launch=False):
    shape = synth.SEVEN_B.replace(d_model=d, n_heads=heads, d_ff=d_ff, n_layers=1, n_prompts=1, n_nodes=2, tree_widths=None, vocab=1024, logit_lo=0,
                                  logit_hi=1024, grid_h=32, grid_w=32, prefix_len=1, prefix_kind=synth.PREFIX_CLASS)
    pair = gc.Pair(shape, gain_jitter=0.1, shadow=True, sample=[0], norm_mode=norm_mode)
    with gc.layer_launches(pair, one_launch):
        pair.prefill(n_forced=tokens - 1)
    raw, _, _ = pair.gpu_logits()
    diff = raw[pair.rows(), 0] - pair.oracle.prefill_logits
    err = float(np.abs(diff).max())
    print("prefill", d, tokens, "logit error", err, "floor", pair.floor)
    assert err <= gc.logit_tol(shape, pair.floor, pair.fused), (err, pair.floor)
    assert gc.rms(diff) <= gc.logit_rms_tol(shape, pair.floor_rms, pair.fused)
    gc.check_kv(pair, 0, tokens, "prefill", prompts=[0])
    pair.close()
