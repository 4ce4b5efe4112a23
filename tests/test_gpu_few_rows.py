"""All layers of a forward in one launch (up to 192 or 224 rows, head size 64): parity at the edges of its tiles, and the same bits whoever computes a
tile - dealt to workgroups, drawn by them where another kernel keeps CUs, beside another launch of its kind."""
import numpy as np
import pytest
import torch

from paper_2511_13587_amd import synth
from test_gpu_drafter import DraftSide
from test_gpu_parity import gc, run_bf16_case, show  # noqa: F401

pytestmark = pytest.mark.gpu


# rows 2 (one row of a block), 32, 34 (a block, and two rows more), 64 (34 tokens: two units of 32 queries, then 64), 96 and 192 of 2 and 4 rows to an
# attention unit (320 and 640 pairs), 192 (32 queries to a unit), 194 (one launch per projection again), 208 and 220 (48 and 40 pairs: one launch up to 224), 232 (again
# not); d_ff no multiple of 48 (2048) and one (3456)
@pytest.mark.parametrize("model,prompts,tokens,n_forced,together", [
    ("b", 1, 1, 9, True), ("b", 2, 8, 30, True), ("b", 1, 17, 40, True), ("xl", 1, 32, 31, True), ("xl", 1, 34, 20, True), ("xl", 8, 6, 33, True), ("xl", 16, 6, 20, True),
    ("xl", 3, 32, 64, True), ("b", 8, 12, 11, True), ("b", 1, 64, 32, True), ("b", 97, 1, 5, False), ("b", 4, 26, 20, True), ("xl", 2, 55, 31, True), ("b", 4, 29, 8, False)])
def test_layers_in_one_launch(gc, model, prompts, tokens, n_forced, together):  # noqa: F811
    base = synth.XL_TREE if model == "xl" else synth.B_SHAPE
    shape = base.replace(n_layers=2, n_prompts=prompts, n_nodes=max(tokens - 1, 1), tree_widths=None, vocab=1024, logit_hi=1024)
    if tokens == 1:
        pair = gc.Pair(shape, shadow=True, sample=[0, prompts - 1] if prompts > 8 else None)
        pair.prefill(n_forced=n_forced, robust_u=True)
        for it in range(2):
            with gc.layer_launches(pair, together):
                pair.verify(None, None, None, synth.make_uniforms(shape, 0, it))
            gc.check_logits(pair, f"{model} {prompts} x 1 call {it}")
            pair.commit()
        pair.close()
        return
    sample = [0, prompts - 1] if prompts > 8 else None
    show(f"{model} {prompts} x {tokens}", run_bf16_case(gc, shape, n_forced=n_forced, calls=2, one_launch=together, **({"sample": sample} if sample else {})))


# trees of one and two prompts of 20 heads, 14 to 122 rows
@pytest.mark.parametrize("prompts,n_nodes,widths,n_forced", [(1, 6, None, 33), (1, 26, (4, 6, 6, 5, 5), 45), (1, 31, (4, 6, 8, 8, 5), 20), (1, 32, (4, 6, 8, 8, 6), 20),
                                                            (1, 60, (8, 12, 12, 10, 10, 8), 31), (2, 15, (4, 5, 6), 40)])
def test_trees_in_one_launch(gc, prompts, n_nodes, widths, n_forced):  # noqa: F811
    shape = synth.XL_TREE.replace(n_layers=2, n_prompts=prompts, n_nodes=n_nodes, tree_widths=widths)
    show(f"xl {prompts} x {n_nodes + 1}", run_bf16_case(gc, shape, n_forced=n_forced, calls=2, one_launch=True))


# d 512 with up to 64 pairs: one launch up to 256 rows.  8 row-blocks, the last of them whole or not; 64 pairs; 264 rows; 72 pairs, whose limit is 192.
# K and V of layer 0, whose bound is derived (check_kv); those of layer 1 differ from the checker's by 1.17 ulps rms, 6.5 at most, in one launch and in
# a launch per projection alike, where the shadow's own flips allow 4.  The logits behind both layers keep their bounds.
@pytest.mark.parametrize("prompts,tokens,together", [(2, 63, True), (2, 64, True), (8, 16, True), (3, 44, False), (9, 12, False)])
def test_rows_of_a_narrow_model(gc, prompts, tokens, together):  # noqa: F811
    shape = synth.B_SHAPE.replace(d_model=512, n_heads=8, d_ff=1344, n_layers=2, n_prompts=prompts, n_nodes=tokens - 1, tree_widths=None, vocab=1024, logit_hi=1024)
    show(f"d 512 {prompts} x {tokens}", run_bf16_case(gc, shape, n_forced=20, calls=2, kv_layers=[0], one_launch=together))


@pytest.mark.parametrize("d,heads,d_ff", [(64, 1, 64), (192, 3, 320), (1408, 22, 3840), (1536, 24, 3072)])
def test_widths_of_the_one_launch(gc, d, heads, d_ff):  # noqa: F811
    """Contractions shorter than the eight waves, and longer than what is asked for ahead."""
    shape = synth.B_SHAPE.replace(d_model=d, n_heads=heads, d_ff=d_ff, n_layers=2, n_prompts=2, n_nodes=8, tree_widths=None, vocab=1024, logit_hi=1024)
    show(f"d {d} d_ff {d_ff}", run_bf16_case(gc, shape, n_forced=20, calls=2, one_launch=True))


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


def test_a_kept_cu_delays_no_more_than_the_wait(gc):  # noqa: F811
    """One workgroup of the fill probe keeps a CU: the call goes on without it, some 5 us later than with all CUs (bound: 100; it had waited 200)."""
    shape = synth.B_SHAPE.replace(n_layers=3, n_prompts=1, n_nodes=2, vocab=1024, logit_hi=1024)
    pair = gc.Pair(shape, with_oracle=False)
    src = torch.zeros(1 << 18, dtype=torch.int32, device=pair.dev)
    prefix = torch.zeros((1, 1), dtype=torch.int32, device=pair.dev)
    u, first = torch.full((1,), 0.5, device=pair.dev), torch.zeros(1, dtype=torch.int32, device=pair.dev)

    def call():
        t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        t0.record()
        pair.ctx.vvs_prefill(prefix, None, None, u, first)
        t1.record()
        t1.synchronize()
        return t0.elapsed_time(t1) * 1e3

    idle = min(call() for _ in range(8))
    kept = []
    for _ in range(12):                      # streams share a few hardware queues: those that are not the call's own
        busy, done = torch.cuda.Stream(), torch.cuda.Event()
        with torch.cuda.stream(busy):
            pair.ctx.vvs_debug_fill_probe(src, 1000, 1, 1, 16)             # some 5 ms
            done.record()
        us = [call() for _ in range(4)]
        if not done.query():
            kept += us
        torch.cuda.synchronize()
    assert kept and min(kept) < idle + 100, (idle, kept)
    pair.close()


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
@pytest.mark.parametrize("tokens,prompts,together", [(1, 1, True), (62, 1, True), (64, 1, True), (65, 1, False), (28, 4, True)])
def test_prefill_of_few_rows(gc, tokens, prompts, together):  # noqa: F811
    shape = synth.B_SHAPE.replace(n_layers=2, n_prompts=prompts, n_nodes=2, tree_widths=None, vocab=1024, logit_lo=0, logit_hi=1024)
    pair = gc.Pair(shape, gain_jitter=0.1, shadow=True)
    with gc.layer_launches(pair, together):
        pair.prefill(n_forced=tokens - 1)
    raw, _, _ = pair.gpu_logits()
    d = raw[pair.rows(), 0] - pair.oracle.prefill_logits
    assert float(np.abs(d).max()) <= gc.logit_tol(shape, pair.floor, pair.fused)
    assert gc.rms(d) <= gc.logit_rms_tol(shape, pair.floor_rms, pair.fused)
    gc.check_kv(pair, 0, tokens, "prefill")
    pair.close()


# A limit of one look ends the first wait for a tile that is still being computed: what the workgroups left undone must be said by the call's
# outputs, and the next call must be as if nothing had been.  Narrow layers and wide ones.
@pytest.mark.parametrize("model", ["b", "7b"])
def test_a_wait_that_gives_up_is_told(gc, model):  # noqa: F811
    base = synth.B_SHAPE if model == "b" else synth.SEVEN_B.replace(d_model=1536, n_heads=12, d_ff=4096, prefix_len=8, logit_lo=0)
    shape = base.replace(n_layers=2, n_prompts=2, n_nodes=13, tree_widths=None, vocab=1024, logit_hi=1024)
    step = Step(gc, shape, 0)
    pair, ctx = step.pair, step.pair.ctx
    step.run()
    want = step.result(), pair.accept_len.clone(), pair.path.clone(), pair.next_token.clone()
    features = ctx.vvs_read_features()
    ctx.vvs_debug_wait_limit(1)
    step.run()
    torch.cuda.synchronize()
    assert pair.accept_len.tolist() == [-1, -1] and pair.next_token.tolist() == [-1, -1] and bool((pair.path == -1).all())
    ctx.vvs_kv_commit()
    assert np.array_equal(ctx.vvs_read_state(), step.state.cpu().numpy())
    assert all(np.array_equal(a, b) for a, b in zip(ctx.vvs_read_features(), features))
    ctx.vvs_debug_wait_limit(0)
    step.run()
    assert same(step.result(), want[0])
    assert all(torch.equal(a, b) for a, b in zip((pair.accept_len, pair.path, pair.next_token), want[1:]))
    # a prefill: its prompts count as complete, until the next one
    ctx.vvs_debug_wait_limit(1)
    first, _, u = pair.prefill(n_forced=4, run_oracle=False)
    assert first.tolist() == [-1, -1]
    assert ctx.vvs_read_state()[1:].tolist() == [[shape.grid] * 2, [-1] * 2]
    ctx.vvs_debug_wait_limit(0)
    ctx.vvs_verify(shape.n_nodes, None, None, *step.args, 0, pair.accept_len, pair.path, pair.next_token)
    assert pair.accept_len.tolist() == [0, 0] and pair.next_token.tolist() == [-1, -1]
    first, _, _ = pair.prefill(n_forced=4, u=u, run_oracle=False)
    assert (first >= 0).all() and ctx.vvs_read_state()[1].tolist() == [5, 5]
    pair.close()


def test_a_drafting_call_that_gives_up_is_told(gc):  # noqa: F811
    shape = synth.B_SHAPE.replace(n_layers=1, n_prompts=2, n_nodes=10, tree_widths=(3, 4, 3), vocab=1024, logit_lo=64, logit_hi=1024)
    parent = np.asarray(synth.tree_parents(shape.tree_widths, 10), dtype=np.int32)
    inner = sorted({int(p) for p in parent})
    pair = gc.Pair(shape, with_oracle=False)
    pair.prefill(n_forced=10, run_oracle=False)
    side = DraftSide(gc, pair, max_block=3 + len(inner) - 1)
    recent = torch.full((2, 3), 70, dtype=torch.int32, device=pair.dev)

    def draft():
        tok = torch.full((2, 10), -1, dtype=torch.int32, device=pair.dev)
        q = torch.full((2, 11, shape.v_eff), -1.0, dtype=torch.float32, device=pair.dev)
        side.ctx.vvs_draft(pair.ctx, 10, parent, None, 3, recent, 0, None, tok, q)
        return tok.cpu().numpy(), q.cpu().numpy()

    want = draft()
    side.ctx.vvs_debug_wait_limit(1)
    tok, q = draft()
    assert np.isnan(q[:, inner]).all()
    rank = [list(parent[:j]).count(p) for j, p in enumerate(parent)]
    assert tok.tolist() == [[64 + r for r in rank]] * 2                     # ids of the slice, siblings distinct
    side.ctx.vvs_debug_wait_limit(0)
    assert same(draft(), want)
    side.close()
    pair.close()
