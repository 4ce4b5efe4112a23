"""A drafting call computes every block token once, level by level: its logits stand afterwards for the pairs and every expanded
node, and the distributions handed out are the softmax of them."""
import numpy as np
import pytest
import torch

from paper_2511_13587_amd import synth
from test_gpu_drafter import DraftSide, gc  # noqa: F401

pytestmark = pytest.mark.gpu


# a chain (one node a level), a tree whose levels grow, a single node (level 0 alone); head sizes 32 (fp32) and 64, up to 64 block tokens
@pytest.mark.parametrize("model,k,parent", [("tiny", 5, None), ("tiny", 1, None), ("tiny", 2, (0,)), ("xl", 5, (4, 6, 6, 5, 5)), ("b", 3, None),
                                            ("b", 5, (8, 12, 12, 10, 10, 8))])
def test_logits_of_a_drafting_call(gc, model, k, parent):  # noqa: F811
    base = {"tiny": synth.TINY, "xl": synth.XL_TREE.replace(vocab=1024, logit_lo=0, logit_hi=1024), "b": synth.B_SHAPE}[model]
    n = 12 if parent is None else 1 if len(parent) == 1 else sum(parent)
    shape = base.replace(n_layers=1, n_nodes=n, n_prompts=2, tree_widths=None if parent is None or n == 1 else parent)
    par = np.asarray(synth.tree_parents(shape.tree_widths, n), dtype=np.int32)
    pair = gc.Pair(shape, with_oracle=False)
    pair.prefill(n_forced=10, run_oracle=False)
    inner = sorted({int(p) for p in par if p > 0}, key=lambda j: (depth(par, j), j))
    side = DraftSide(gc, pair, max_block=k + len(inner))
    recent = torch.full((2, k), shape.logit_lo + 3, dtype=torch.int32, device=pair.dev)
    tok = torch.full((2, n), -1, dtype=torch.int32, device=pair.dev)
    q = torch.full((2, n + 1, shape.v_eff), -1.0, dtype=torch.float32, device=pair.dev)
    side.ctx.vvs_draft(pair.ctx, n, par, None, k, recent, 0, None, tok, q)
    T = k + len(inner)
    mixed = torch.empty((2, T, shape.v_eff), dtype=torch.float32, device=pair.dev)
    status = gc.vb.lib.vvs_debug_logits(side.ctx.h, None, mixed.data_ptr(), None, torch.cuda.current_stream().cuda_stream)
    assert status == gc.vb.VVS_OK
    assert bool(torch.isfinite(mixed).all())
    want = torch.softmax(mixed.double(), dim=2)
    for place, node in enumerate([0] + inner):
        # fp32 softmax of the same logits: a sum of v_eff terms, each rounded to 2^-24
        err = (q[:, node].double() - want[:, k - 1 + place]).abs().max() / want[:, k - 1 + place].max()
        assert float(err) < 1e-5, (node, float(err))
    assert int(tok.min()) >= shape.logit_lo
    side.close()
    pair.close()


# the selection's forms: up to 4096 ids on 8 waves, 16384 on 16, ids from memory beyond
@pytest.mark.parametrize("ids", [64, 4095, 4096, 4097, 16384, 16385])
def test_children_are_the_likeliest_ids(gc, ids):  # noqa: F811
    shape = synth.TINY.replace(n_layers=1, vocab=ids + 8, logit_lo=8, logit_hi=ids + 8, n_nodes=12, n_prompts=2, tree_widths=(5, 4, 3))
    par = np.asarray(synth.tree_parents(shape.tree_widths, 12), dtype=np.int32)
    pair = gc.Pair(shape, with_oracle=False)
    pair.prefill(n_forced=10, run_oracle=False)
    inner = sorted({int(p) for p in par if p > 0}, key=lambda j: (depth(par, j), j))
    side = DraftSide(gc, pair, max_block=3 + len(inner))
    recent = torch.full((2, 3), 11, dtype=torch.int32, device=pair.dev)
    tok = torch.full((2, 12), -1, dtype=torch.int32, device=pair.dev)
    q = torch.empty((2, 13, ids), dtype=torch.float32, device=pair.dev)
    side.ctx.vvs_draft(pair.ctx, 12, par, None, 3, recent, 0, None, tok, q)
    mixed = torch.empty((2, 3 + len(inner), ids), dtype=torch.float32, device=pair.dev)
    assert gc.vb.lib.vvs_debug_logits(side.ctx.h, None, mixed.data_ptr(), None, torch.cuda.current_stream().cuda_stream) == gc.vb.VVS_OK
    mixed, got = mixed.cpu().numpy(), tok.cpu().numpy()
    for place, node in enumerate([0] + inner):
        kids = [c for c in range(1, 13) if par[c - 1] == node]
        for b in range(2):
            row = mixed[b, 2 + place]
            # both mix the same two logits, one perhaps with a fused multiply-add: a value 2^-22 of the largest beside the next
            assert np.abs(row[got[b, [c - 1 for c in kids]] - 8] - np.sort(row)[::-1][:len(kids)]).max() <= 2.0 ** -22 * np.abs(row).max()
            assert len({int(got[b, c - 1]) for c in kids}) == len(kids)
    side.close()
    pair.close()


def depth(par, j):
    d = 0
    while j:
        j, d = int(par[j - 1]), d + 1
    return d
