"""All layers of a forward in one launch (up to 192 or 224 rows, head size 64): parity at the edges of its tiles, and the same bits whoever computes a
tile - dealt to workgroups, drawn by them where another kernel keeps CUs, beside another launch of its kind."""
import numpy as np
import pytest
import torch

from paper_2511_13587_amd import synth
from test_gpu_parity import gc, run_bf16_case, show  # noqa: F401

pytestmark = pytest.mark.gpu


# rows 2 (one row of a block), 32, 34 (a block, and two rows more), 64 (34 tokens: two units of 32 queries, then 64), 96 and 192 of 2 and 4 rows to an
# attention unit (320 and 640 pairs), 192 (32 queries to a unit), 194 (one launch per projection again), 208 and 220 (48 and 40 pairs: one launch up to 224), 232 (again
# not); d_ff no multiple of 48 (2048) and one (3456)
@pytest.mark.parametrize("model,prompts,tokens,n_forced", [("b", 1, 1, 9), ("b", 2, 8, 30), ("b", 1, 17, 40), ("xl", 1, 32, 31), ("xl", 1, 34, 20), ("xl", 8, 6, 33),
                                                           ("xl", 16, 6, 20), ("xl", 3, 32, 64), ("b", 8, 12, 11), ("b", 1, 64, 32), ("b", 97, 1, 5), ("b", 4, 26, 20), ("xl", 2, 55, 31), ("b", 4, 29, 8)])
def test_layers_in_one_launch(gc, model, prompts, tokens, n_forced):  # noqa: F811
    base = synth.XL_TREE if model == "xl" else synth.B_SHAPE
    shape = base.replace(n_layers=2, n_prompts=prompts, n_nodes=max(tokens - 1, 1), tree_widths=None, vocab=1024, logit_hi=1024)
    if tokens == 1:
        pair = gc.Pair(shape, shadow=True, sample=[0, prompts - 1] if prompts > 8 else None)
        pair.prefill(n_forced=n_forced, robust_u=True)
        for it in range(2):
            pair.verify(None, None, None, synth.make_uniforms(shape, 0, it))
            gc.check_logits(pair, f"{model} {prompts} x 1 call {it}")
            pair.commit()
        pair.close()
        return
    sample = [0, prompts - 1] if prompts > 8 else None
    show(f"{model} {prompts} x {tokens}", run_bf16_case(gc, shape, n_forced=n_forced, calls=2, **({"sample": sample} if sample else {})))


@pytest.mark.parametrize("d,heads,d_ff", [(64, 1, 64), (192, 3, 320), (1408, 22, 3840), (1536, 24, 3072)])
def test_widths_of_the_one_launch(gc, d, heads, d_ff):  # noqa: F811
    """Contractions shorter than the eight waves, and longer than what is asked for ahead."""
    shape = synth.B_SHAPE.replace(d_model=d, n_heads=heads, d_ff=d_ff, n_layers=2, n_prompts=2, n_nodes=8, tree_widths=None, vocab=1024, logit_hi=1024)
    show(f"d {d} d_ff {d_ff}", run_bf16_case(gc, shape, n_forced=20, calls=2))


class Step:
    """A context whose verify call can be repeated, on a stream of its own."""
    def __init__(self, gc, shape, seed):  # noqa: F811
        self.shape, self.stream = shape, torch.cuda.Stream()
        self.pair = gc.Pair(shape, with_oracle=False)
        self.pair.prefill(n_forced=40, run_oracle=False)
        dev, n = self.pair.dev, shape.n_nodes
        q, toks = synth.make_draft(shape, synth.tree_parents(None, n), seed)
        self.args = [torch.from_numpy(x).to(dev) for x in (toks, q, synth.make_uniforms(shape, n, seed))]
        self.state = torch.from_numpy(self.pair.ctx.vvs_read_state()).to(dev)
        torch.cuda.synchronize()

    def run(self):
        with torch.cuda.stream(self.stream):
            self.pair.ctx.vvs_set_state(self.state)
            self.pair.ctx.vvs_verify(self.shape.n_nodes, None, None, *self.args, 0, self.pair.accept_len, self.pair.path, self.pair.next_token)

    def result(self):
        self.stream.synchronize()
        raw = self.pair.ctx.vvs_debug_logits()[0].cpu().numpy().copy()
        k, v = self.pair.ctx.vvs_debug_kv(self.shape.n_layers - 1, 1, int(self.state[0, 0]) + self.shape.n_nodes + 1)
        return raw, k.cpu().numpy().copy(), v.cpu().numpy().copy()


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def test_tiles_drawn_while_another_kernel_keeps_cus(gc):  # noqa: F811
    """200 workgroups of the fill probe hold the LDS of a CU each for longer than the call takes: its workgroups are not all there, and those that
    run draw the tiles.  The probe still being at work when the call is over says that no workgroup waited for those CUs."""
    shape = synth.B_SHAPE.replace(n_layers=3, n_prompts=3, n_nodes=11, vocab=1024, logit_hi=1024)
    step = Step(gc, shape, 0)
    step.run()
    want = step.result()
    src = torch.zeros(1 << 18, dtype=torch.int32, device=step.pair.dev)
    overlapped = False
    for _ in range(8):                       # streams share a few hardware queues: one that is not the call's own
        busy, done = torch.cuda.Stream(), torch.cuda.Event()
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            step.pair.ctx.vvs_debug_fill_probe(src, 4000, 1, 200, 16)      # some 40 ms
            done.record()
        step.run()
        step.stream.synchronize()
        overlapped = overlapped or not done.query()
        assert same(step.result(), want)
        torch.cuda.synchronize()
        if overlapped:
            break
    assert overlapped, "the probe was over before the call: nothing was tested"
    step.run()                                                             # the counters are as before
    assert same(step.result(), want)
    step.pair.close()


def test_two_launches_of_the_kind_at_once(gc):  # noqa: F811
    shapes = [synth.B_SHAPE.replace(n_layers=4, n_prompts=p, n_nodes=n, vocab=1024, logit_hi=1024) for p, n in ((2, 9), (3, 20), (1, 40))]
    steps = [Step(gc, s, i) for i, s in enumerate(shapes)]
    want = []
    for s in steps:
        s.run()
        want.append(s.result())
    for _ in range(10):
        for s in steps:
            s.run()
    for s, w in zip(steps, want):
        assert same(s.result(), w)
    for s in steps:
        s.pair.close()


# 2 rows; 62 and 64 tokens of one prompt (the last that the masks hold), 65 (projections and attention apart again); 224 rows
@pytest.mark.parametrize("tokens,prompts", [(1, 1), (62, 1), (64, 1), (65, 1), (28, 4)])
def test_prefill_of_few_rows(gc, tokens, prompts):  # noqa: F811
    shape = synth.B_SHAPE.replace(n_layers=2, n_prompts=prompts, n_nodes=2, tree_widths=None, vocab=1024, logit_lo=0, logit_hi=1024)
    pair = gc.Pair(shape, gain_jitter=0.1, shadow=True)
    pair.prefill(n_forced=tokens - 1)
    raw, _, _ = pair.gpu_logits()
    d = raw[pair.rows(), 0] - pair.oracle.prefill_logits
    assert float(np.abs(d).max()) <= gc.logit_tol(shape, pair.floor, pair.fused)
    assert gc.rms(d) <= gc.logit_rms_tol(shape, pair.floor_rms, pair.fused)
    gc.check_kv(pair, 0, tokens, "prefill")
    pair.close()
