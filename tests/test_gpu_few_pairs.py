"""GPU parity of verify calls on both sides of the lines between one launch for q/k/v projection and attention and two, with more rows than
take all layers in one launch: few (head, prompt) pairs, pairs that fill their rounds of CUs badly, and the projection on 32 x 32 tiles."""
import pytest

from paper_2511_13587_amd import synth
from test_gpu_parity import gc, run_bf16_case, show  # noqa: F401
from test_gpu_shared_tiles import check_prefill

pytestmark = pytest.mark.gpu


# 32 pairs of d 1024 (240 rows) and 36 of d 1152; 260 pairs of 20 heads (208 rows), 264 of 12.  K and V of layer 0, whose bound is derived (see
# test_projection_and_attention_together_in_rounds: one element in 24192 of the prefilled K of layer 1, d 1152, is 4.75 ulps off where the flips allow 4)
@pytest.mark.parametrize("d,heads,d_ff,prompts,n_nodes,widths,n_forced", [(1024, 16, 2752, 2, 59, (8, 12, 12, 10, 10, 7), 33), (1152, 18, 3072, 2, 57, None, 20),
                                                                         (1280, 20, 3456, 13, 7, (2, 3, 2), 40), (768, 12, 2048, 22, 5, None, 9)])
def test_projection_and_attention_apart(gc, d, heads, d_ff, prompts, n_nodes, widths, n_forced):  # noqa: F811
    shape = synth.B_SHAPE.replace(d_model=d, n_heads=heads, d_ff=d_ff, n_layers=2, n_prompts=prompts, n_nodes=n_nodes, tree_widths=widths)
    assert attention_launches(gc, shape.replace(n_layers=1, vocab=1024, logit_hi=1024)) == 1
    sample = [0, prompts - 1] if prompts > 8 else None
    show(f"d {d} {prompts} x {n_nodes + 1}", run_bf16_case(gc, shape, n_forced=n_forced, calls=2, kv_layers=[0], one_launch=False, **({"sample": sample} if sample else {})))


# 12 heads: up to 256 pairs one round of CUs, whatever the tokens; two and three rounds while pairs and tokens fill 0.665 and 0.89 of them
@pytest.mark.parametrize("prompts,tokens,together", [(21, 1, True), (22, 21, False), (30, 61, True), (30, 60, False), (36, 27, True), (36, 25, False), (42, 32, True),
                                                     (43, 32, False), (60, 32, True), (60, 30, False), (64, 56, False), (64, 57, True), (66, 64, False)])
def test_rounds_of_projection_and_attention_together(gc, prompts, tokens, together):  # noqa: F811
    shape = synth.B_SHAPE.replace(n_layers=1, n_prompts=prompts, n_nodes=tokens - 1, vocab=1024, logit_hi=1024)
    assert attention_launches(gc, shape) == (0 if together else 1)


def attention_launches(gc, shape):  # noqa: F811
    """Attention launches of a verify call of one layer."""
    n = shape.n_nodes
    pair = gc.Pair(shape, with_oracle=False)
    pair.prefill(n_forced=3, run_oracle=False)
    q, toks = synth.make_draft(shape, synth.tree_parents(None, n), 0) if n else (None, None)
    pair.ctx.vvs_timing_enable(True)
    pair.verify(None, toks, q, synth.make_uniforms(shape, n, 0), run_oracle=False)
    n_attention, _ = pair.ctx.vvs_timing_read(gc.vb.VVS_K_ATTENTION)
    pair.ctx.vvs_timing_enable(False)
    pair.close()
    return n_attention


# Two rounds, the second two thirds full, and three.  K and V of layer 0, whose bound is derived (check_kv): deeper ones add 3 x the shadow's own
# change, which is the few roundings that happen to flip there, and the prefilled K of prompt 59 holds one element in 16128 at 5 ulps - here and with
# the projection and attention apart alike - where those flips allow 4.75.  The logits behind both layers keep their bounds.
@pytest.mark.parametrize("prompts,n_nodes,widths", [(36, 26, (4, 6, 6, 5, 5)), (60, 31, (4, 6, 8, 8, 5))])
def test_projection_and_attention_together_in_rounds(gc, prompts, n_nodes, widths):  # noqa: F811
    shape = synth.B_SHAPE.replace(n_layers=2, n_prompts=prompts, n_nodes=n_nodes, tree_widths=widths)
    show(f"b {prompts} x {n_nodes + 1}", run_bf16_case(gc, shape, n_forced=20, calls=2, sample=[0, prompts - 1], kv_layers=[0]))


# q/k/v on 32 x 32 tiles with positions and rotary factors from memory instead of LDS (head size 128), and behind a normalisation of its own:
# d_model, heads, d_ff, prompts, tokens, norm mode; 18 and 54 rows (a row-block and a part of one, two), 144 (more than take all layers in one launch)
SMALL_TILES = [(1024, 8, 2752, 1, 9, 0), (1024, 8, 2752, 1, 27, 0), (512, 4, 1408, 3, 24, 1), (512, 8, 1408, 3, 24, 1)]


@pytest.mark.parametrize("d,heads,d_ff,prompts,tokens,norm_mode", SMALL_TILES)
def test_small_tiles_of_the_projection(gc, d, heads, d_ff, prompts, tokens, norm_mode):  # noqa: F811
    shape = synth.SEVEN_B.replace(d_model=d, n_heads=heads, d_ff=d_ff, n_layers=2, n_prompts=prompts, n_nodes=tokens - 1, tree_widths=None, vocab=1024,
                                  logit_lo=0, logit_hi=1024)
    show(f"d {d} heads {heads} tokens {tokens}", run_bf16_case(gc, shape, n_forced=40, calls=2, norm_mode=norm_mode, one_launch=False))


def test_small_tiles_of_a_prefill(gc):  # noqa: F811
    """... and at head size 64 without one, which only a prefill of more tokens than the masks hold takes (140 rows of d 512)."""
    check_prefill(gc, 512, 8, 1408, 70)
