"""The forms of the acceptance kernel by slice width and number of nodes, against the oracle's acceptance procedure on given logits."""
import numpy as np
import pytest
import torch

from oracle import vvs_oracle as vo
from paper_2511_13587_amd import binding as vb
from paper_2511_13587_amd import synth

pytestmark = pytest.mark.gpu


# ids: 4 waves up to 4096, then 16 up to 16384 ids in registers; nodes: up to 1280 (20 x 64), with the relaxed rule up to 576 (9 x 64), in workgroups of 1024
# threads, more (21 x 61, 10 x 64) of 512; 16381 ids: rows that do not start on 16 bytes, in both
@pytest.mark.parametrize("ids,prompts,nodes", [(1024, 1, 4), (4096, 3, 12), (4160, 3, 12), (16384, 4, 63), (16384, 9, 63), (16384, 10, 63), (16384, 16, 63), (16384, 20, 63),
                                               (16384, 21, 60), (16320, 21, 62), (16320, 5, 60), (16381, 3, 20), (16381, 21, 61), (16448, 2, 7)])
@pytest.mark.parametrize("mode", [vb.VVS_STRICT, vb.VVS_RELAXED])
def test_forms(ids, prompts, nodes, mode):
    shape = synth.TINY.replace(n_layers=1, vocab=ids, logit_hi=ids, n_prompts=prompts, n_nodes=nodes, relax_k=8, relax_delta=0.2)
    ctx = vb.Context(vb.make_config(shape))
    g = torch.Generator("cuda")
    g.manual_seed(ids + prompts)
    normal = lambda *dims: torch.empty(dims, device="cuda").normal_(generator=g)   # noqa: E731
    nbr = torch.randint(0, ids, (ids, 8), generator=g, device="cuda", dtype=torch.int32)
    ctx.vvs_set_neighbors(nbr)
    parent = synth.tree_parents((2, nodes - 2), nodes)
    logits = normal(prompts, 2, nodes + 1, ids)
    q = torch.softmax(logits[:, 0] + normal(prompts, nodes + 1, ids), dim=2)
    rank = [list(parent[:j]).count(p) for j, p in enumerate(parent)]
    picks = torch.multinomial(q.view(-1, ids), max(rank) + 1, generator=g).view(prompts, nodes + 1, -1)
    tokens = picks[:, list(map(int, parent)), rank].to(torch.int32).contiguous()
    u = torch.rand((prompts, nodes + 1, 2), generator=g, device="cuda")
    a, path, nxt = (torch.zeros(dims, dtype=torch.int32, device="cuda") for dims in (prompts, (prompts, vb.VVS_MAX_T), prompts))
    mixed = (logits[:, 1] + shape.cfg_scale * (logits[:, 0] - logits[:, 1])).double().cpu().numpy()
    p = np.exp(mixed - mixed.max(axis=2, keepdims=True))
    p /= p.sum(axis=2, keepdims=True)
    host = [x.cpu().numpy() for x in (q.double(), tokens, u, nbr)]
    compared = 0
    for _ in range(3):                                   # the counters of the walk are as they were
        ctx.vvs_accept_from_logits(nodes, parent, None, logits, tokens, q, u, mode, a, path, nxt)
        for b in range(prompts):
            tr = {}
            want = vo.decide(p[b], host[0][b], host[1][b], parent, host[2][b], nodes, mode, host[3], 8, 0.2, trace=tr)
            # sums of up to 16448 ids in 32 bits: 1e-5 of a threshold or of an edge of the drawn interval may fall either way
            if min(tr["accept_margin"], tr["relax_margin"], np.abs(tr["term_cdf"] - tr["term_u"]).min()) < 1e-5:
                continue
            compared += 1
            assert (int(a[b]), path[b][:int(a[b]) + 1].tolist(), int(nxt[b])) == (want[0], list(want[1]), want[2])
    assert compared * 2 > 3 * prompts, "hardly any outcome was clear of its thresholds"
    ctx.close()
