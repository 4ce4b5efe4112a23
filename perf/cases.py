"""The cases this library's performance is measured on, as calls through its Python binding.

A case is one of four things a program around the library does over and over, on one of the model shapes of
paper_2511_13587_amd.synth (random-init weights; everything else a function of the seed):

  step     one target pass of a decoding loop: vvs_verify (or vvs_verify_post) over a drafted chain or tree, then
           vvs_kv_commit.  The call starts from a saved per-prompt state (vvs_set_state), so that it can be repeated.
  prefill  vvs_prefill of the condition prefix and, where an image is taken up again, of its first tokens.
  draft    vvs_draft: the one-block drafter fills a candidate tree from the target's cached features; the tokens are the
           caller's own samples (d_given_tokens), the distributions the drafter's.
  accept   vvs_accept_from_logits: mix, softmax, accept / resample on logits that another program computed.
  loop     one round of the whole loop in fp32 on the reference shape: draft (greedy), path similarity, verify, commit.

What the outputs hold.  Accept lengths, paths and tokens are compared as whole numbers.  The token drawn at the end of a
bf16 pass is left out there: with logit noise at the level of the bf16 roundings (about 1e-2, times 14 through the guidance
mix) the inverse CDF gives a neighbouring token for one prompt in ten, whoever computes it.  The bf16 passes return
the raw logits of every scored node, the path and the KV cache after the commit; the drawn tokens are compared where
the logits are given (accept) or fp32 (loop).  For the same reason the accept tests of these passes are clear: the uniforms of the
nodes to accept are 0, the other drafted tokens are sure of themselves and wrong (the drafter gives each more than half of
what its elder siblings left, the target hardly anything), so that accept lengths are those drawn in prepare(), with the
paper's means (1.22 tokens per pass with strict acceptance, 2.27 relaxed)."""
import math
import random

import numpy as np
import torch

from paper_2511_13587_amd import binding as vb
from paper_2511_13587_amd import synth

MODELS = {"tiny": synth.TINY, "b": synth.B_SHAPE, "xl": synth.XL_TREE, "7b": synth.SEVEN_B}
RELAX_K, RELAX_DELTA = synth.XL_STRESS.relax_k, synth.XL_STRESS.relax_delta


# ------------------------------------------------------------------------------------------------ the cases
def _step(name, model, prompts, nodes, tree, cached, ragged=False, post=0, relaxed=False):
    return {"name": name, "path": "step", "model": model, "prompts": prompts, "nodes": nodes, "tree": tree, "post": post,
            "cached": cached, "ragged": ragged, "relaxed": relaxed}


def listed():
    return [
        # the smallest work there is: the fp32 reference shape, one prompt, chain of 4, the whole loop - launches and host time only
        {"name": "loop_tiny_fp32", "path": "loop", "model": "tiny", "prompts": 1, "nodes": 4, "tree": False, "cached": 32, "context": 5},
        # the small bf16 model as it is served: class-conditional, a chain of 5, half way through its 16 x 16 image
        _step("step_b_chain5_x4", "b", 4, 5, False, 128),
        # one image for one user (how the paper times whole images): 2 rows, 26-node tree
        _step("step_xl_tree26_x1", "xl", 1, 26, True, 288),
        # the benchmark's workload
        _step("step_xl_tree26_x8", "xl", 8, 26, True, 288),
        # an odd batch some steps later: ragged lengths near the end of the image, relaxed rule, three unverified tokens riding in front
        _step("step_xl_post3_x5", "xl", 5, 26, True, 500, ragged=True, post=3, relaxed=True),
        # the largest call: 64 rows of 61 tokens, relaxed acceptance
        _step("step_xl_tree60_x32", "xl", 32, 60, True, 288, relaxed=True),
        # weight streaming: the 7B shape with a chain of 6 for two prompts
        _step("step_7b_chain6_x2", "7b", 2, 6, False, 512),
        # the same model with a tree: head size 128, 126 ragged rows
        _step("step_7b_tree20_x3", "7b", 3, 20, True, 300, ragged=True),
        # the caption prefix of a new batch of images
        {"name": "prefill_xl_x8", "path": "prefill", "model": "xl", "prompts": 8, "forced": 0},
        # the 7B shape's prefix, and an image taken up again after two of its rows
        {"name": "prefill_7b_x2", "path": "prefill", "model": "7b", "prompts": 2, "forced": 33},
        # the draft side at the benchmark's workload, all five cached features as context
        {"name": "draft_xl_tree26_x8", "path": "draft", "model": "xl", "prompts": 8, "nodes": 26, "tree": True, "cached": 288, "context": 5},
        # the acceptance stage alone at the benchmark's width
        {"name": "accept_xl_tree26_x8", "path": "accept", "model": "xl", "prompts": 8, "nodes": 26, "tree": True, "relaxed": False},
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    largest = max(_seconds(c) for c in listed())
    while True:
        path = rng.choices(["step", "prefill", "draft", "accept", "loop"], [10, 3, 2, 2, 1])[0]
        if path == "loop":
            nodes = _log_int(rng, 1, 24)
            c = {"path": path, "model": "tiny", "prompts": _log_int(rng, 1, 6), "nodes": nodes, "tree": nodes > 4 and rng.random() < 0.5,
                 "cached": rng.randint(8, 63 - nodes - 2), "context": rng.randint(1, 5)}
        elif path == "prefill":
            model = rng.choice(["b", "xl", "xl", "7b"])
            c = {"path": path, "model": model, "prompts": _log_int(rng, 1, 6 if model == "7b" else 32),
                 "forced": rng.choice([0, _log_int(rng, 1, MODELS[model].grid - 1)])}
        elif path == "draft":
            nodes = _log_int(rng, 2, 60)
            c = {"path": path, "model": rng.choice(["b", "xl"]), "prompts": _log_int(rng, 1, 32), "nodes": nodes,
                 "tree": nodes > 8 or rng.random() < 0.5, "cached": rng.randint(8, 180), "context": rng.randint(1, 5)}
        elif path == "accept":
            c = {"path": path, "model": rng.choice(["b", "xl", "7b"]), "prompts": _log_int(rng, 1, 32), "nodes": rng.choice([0, _log_int(rng, 1, 63)])}
            most = 31 if c["model"] == "7b" else 63
            c["nodes"] = min(c["nodes"], most)
            c.update(tree=c["nodes"] > 8 or rng.random() < 0.5, relaxed=c["model"] != "7b" and rng.random() < 0.5)
        else:
            model = rng.choice(["b", "xl", "xl", "7b"])
            wide = model == "7b"
            post = rng.choice([0, 0, rng.randint(1, 5)])
            nodes = rng.choice([0] + 5 * [_log_int(rng, 1, (31 if wide else 63) - post)])
            relaxed = not wide and rng.random() < 0.4
            c = {"path": path, "model": model, "prompts": _log_int(rng, 1, 6 if wide else 32), "nodes": nodes,
                 "tree": nodes > 8 or rng.random() < 0.5, "post": post, "cached": rng.randint(8, MODELS[model].grid - nodes - post - 2),
                 "ragged": rng.random() < 0.5, "relaxed": relaxed}
        if _seconds(c) <= largest:
            return c


# ------------------------------------------------------------------------------------------------ sizes
def _shape(case):
    s = MODELS[case["model"]].replace(n_prompts=case["prompts"], n_nodes=case.get("nodes", 0) + case.get("post", 0))
    return s.replace(relax_k=RELAX_K, relax_delta=RELAX_DELTA) if case.get("relaxed") else s


def _parents(case):
    """Parent array of the whole call (the post-verified chain in front), or None for a chain.  Trees have the per-depth
    profile of the benchmark's 26-node tree (of its 60-node tree from 44 nodes on)."""
    n, post = case["nodes"], case.get("post", 0)
    if not case["tree"] or n < 2:
        return None
    profile = (synth.XL_STRESS if n >= 44 else synth.XL_TREE).tree_widths
    ends = [round(n * c / sum(profile)) for c in np.cumsum(profile)]
    widths = [b - a for a, b in zip([0] + ends[:-1], ends) if b > a]
    tree = synth.tree_parents(tuple(widths), n)
    return np.asarray(list(range(post)) + [int(p) + post for p in tree], dtype=np.int32)


def _expanded(parent, n):
    """Nodes that have children, root excluded."""
    return n - 1 if parent is None else len({int(p) for p in parent if p > 0})


def work(case):
    s = _shape(case)
    d, f, layers, v, r, b = s.d_model, s.d_ff, s.n_layers, s.v_eff, s.n_rows, s.n_prompts
    e = 2 if s.dtype == synth.DTYPE_BF16 else 4
    block = 4 * d * d + 3 * d * f
    if case["path"] == "prefill":
        n = s.prefix_len + case["forced"]
        return {"bytes": e * (layers * block + d * v + r * n * d) + e * 2 * r * layers * n * d + 4 * r * v,
                "flops": 2 * r * (n * layers * block + d * v) + 2 * r * layers * n * n * d}
    parent, t = _parents(case), s.n_nodes + 1
    inner = (_expanded(parent, s.n_nodes) + 1) if s.n_nodes else 0        # nodes whose draft row is used
    accept = {"bytes": 4 * v * b * inner, "flops": 10 * b * t * v}
    if case["path"] == "accept":
        return {"bytes": accept["bytes"] + 4 * r * t * v, "flops": accept["flops"]}
    tokens = case.get("context", 0) + inner - 1
    draft = {"bytes": e * (block + 2 * d * d + d * v + r * tokens * 2 * d) + 4 * b * t * v,
             "flops": 2 * r * (tokens * (block + 2 * d * d) + inner * d * v)}
    if case["path"] == "draft":
        return draft
    n = s.prefix_len + case["cached"]
    step = {"bytes": e * (layers * block + d * v + r * t * d) + e * 2 * r * layers * (n + t) * d + 4 * r * t * v + accept["bytes"],
            "flops": 2 * r * t * (layers * block + d * v) + 4 * r * layers * t * (n + t) * d + accept["flops"]}
    if case["path"] == "loop":
        return {k: step[k] + draft[k] for k in step}
    return step


def _seconds(case):
    w = work(case)
    return max(w["bytes"] / 8e12, w["flops"] / 2.5e15)


def tolerance(case):
    if case["path"] == "accept":
        return {"rel": 1e-5, "differ": 0.01}           # whole numbers; a draw on the very edge may fall either way
    if case["path"] == "loop":
        return {"rel": 5e-5, "differ": 0.01}           # fp32 sums of up to 344 terms through three blocks and two softmaxes
    # bf16 operands: the roundings of a layer's operands move the logits by about 0.5 % of their size, and through many
    # layers each rounding that falls the other way moves all that follow
    return {"rel": 0.01 if MODELS[case["model"]].n_layers <= 12 else 0.025, "max": 0.5, "differ": 0.01}


# ------------------------------------------------------------------------------------------------ inputs
class _Maker:
    def __init__(self, seed):
        self.g = torch.Generator("cuda")
        self.g.manual_seed(int(seed))

    def normal(self, dims, dtype=torch.float32, std=1.0, mean=0.0):
        return torch.empty(dims, dtype=dtype, device="cuda").normal_(mean, std, generator=self.g)

    def ids(self, lo, hi, dims):
        return torch.randint(lo, hi, dims, generator=self.g, device="cuda", dtype=torch.int32)

    def uniform(self, dims):
        return torch.rand(dims, generator=self.g, device="cuda")


def _dtype(s):
    return torch.bfloat16 if s.dtype == synth.DTYPE_BF16 else torch.float32


def _weights(mk, s, names):
    dims = dict.fromkeys(names)
    for n in names:
        dims[n] = (2 * s.d_model, s.d_model) if n == "fc" else synth.weight_dims(s, n)
    return {n: mk.normal(dims[n], _dtype(s), 0.16 if n == "fc" else 0.02) if len(dims[n]) > 1 else mk.normal(dims[n], _dtype(s), 0.1, 1.0)
            for n in names}


def _target(mk, s):
    ctx = vb.Context(vb.make_config(s))
    names = synth.weight_names(s)
    if s.prefix_kind == synth.PREFIX_DENSE:
        names = [n for n in names if n != "prefix_embed"]
    w = _weights(mk, s, names)
    ctx.vvs_load_weights([w.get(n) for n in synth.weight_names(s)])
    if s.relax_k:
        code = torch.nn.functional.normalize(mk.normal((s.vocab, 8)), dim=1)
        ctx.vvs_set_neighbors((code @ code.T).fill_diagonal_(-2.0).topk(s.relax_k, dim=1).indices.to(torch.int32).contiguous())
    return ctx, w


def _prefix(mk, s):
    if s.prefix_kind == synth.PREFIX_CLASS:
        return mk.ids(0, s.n_classes, (s.n_prompts, s.prefix_len)), None
    return mk.normal((s.n_prompts, s.prefix_len, s.d_model), _dtype(s)), mk.normal((s.prefix_len, s.d_model), _dtype(s))


def _start(mk, s, ctx, cached, ragged):
    """Prefills `cached` image tokens of every prompt; the state int32 [3, B] of prompts that hold that many (ragged: up to 96 fewer)."""
    first = torch.zeros(s.n_prompts, dtype=torch.int32, device="cuda")
    pc, pu = _prefix(mk, s)
    ctx.vvs_prefill(pc, pu, mk.ids(s.logit_lo, s.logit_hi, (s.n_prompts, cached)), mk.uniform((s.n_prompts,)), first)
    held = torch.full((s.n_prompts,), cached, dtype=torch.int32, device="cuda")
    if ragged:
        held = held - mk.ids(0, min(96, cached - 1) + 1, (s.n_prompts,))
    return torch.stack([held + s.prefix_len, held + 1, mk.ids(s.logit_lo, s.logit_hi, (s.n_prompts,))]).contiguous()


def _draft(mk, s, parent, near=None, noise=1.0):
    """Draft distributions [B, T, V] and tokens [B, N], children drawn without replacement.  near: target logits that the
    distributions resemble, up to the noise; else they resemble nothing, and the drafted children hold most of them: the c-th
    child 0.6 of what the ones before it left."""
    b, n, v = s.n_prompts, s.n_nodes, s.v_eff
    logits = mk.normal((b, n + 1, v), std=s.draft_std) if near is None else near
    q = torch.softmax(logits + noise * mk.normal((b, n + 1, v)), dim=2)
    par = list(range(n)) if parent is None else [int(p) for p in parent]
    rank = [par[:j].count(p) for j, p in enumerate(par)]
    picks = torch.multinomial(q.view(-1, v) + 1e-30, max(rank) + 1, generator=mk.g).view(b, n + 1, -1)
    tokens = picks[:, par, rank]
    if near is None:
        count = torch.tensor([par.count(j) for j in range(n + 1)], device="cuda")
        q *= (0.4 ** count).view(1, -1, 1)
        share = torch.tensor([0.6 * 0.4 ** k for k in rank], device="cuda").expand(b, n)
        q[torch.arange(b, device="cuda").view(b, 1), torch.tensor(par, device="cuda").view(1, n), tokens] += share
    return q, (tokens + s.logit_lo).to(torch.int32).contiguous()


def _outcome(s):
    b = s.n_prompts
    return {"accept_len": torch.zeros(b, dtype=torch.int32, device="cuda"), "path": torch.zeros((b, vb.VVS_MAX_T), dtype=torch.int32, device="cuda"),
            "next": torch.zeros(b, dtype=torch.int32, device="cuda")}


def _clear_uniforms(mk, s, parent, seed, post, relaxed):
    """Uniforms [B, T, 2] with 0 for the nodes to accept: first children from the root (behind the post-verified tokens) down,
    as many as a geometric draw with the paper's mean says.  The others are at least 1/2: times the drafter's 0.6 that is more
    than the 0.2 the relaxed rule may absorb."""
    u = mk.uniform((s.n_prompts, s.n_nodes + 1, 2))
    u[:, :, 0] = 0.5 + 0.5 * u[:, :, 0]
    mean, rng = (1.27 if relaxed else 0.22), random.Random(int(seed))
    par = list(range(s.n_nodes)) if parent is None else [int(p) for p in parent]
    rows, cols = [], []
    for b in range(s.n_prompts):
        node = post
        while rng.random() < mean / (1 + mean) and node in par:
            node = par.index(node) + 1
            rows.append(b)
            cols.append(node)
    u[rows, cols, 0] = 0.0
    return u


def prepare(case, seed):
    mk, s, path = _Maker(seed), _shape(case), case["path"]
    st = {"path": path, "n": s.n_nodes, "mode": vb.VVS_RELAXED if case.get("relaxed") else vb.VVS_STRICT}
    if path == "accept":
        parent = _parents(case)
        st["ctx"] = ctx = vb.Context(vb.make_config(s.replace(n_layers=1)))
        if s.relax_k:
            code = torch.nn.functional.normalize(mk.normal((s.vocab, 8)), dim=1)
            ctx.vvs_set_neighbors((code @ code.T).fill_diagonal_(-2.0).topk(s.relax_k, dim=1).indices.to(torch.int32).contiguous())
        logits = mk.normal((s.n_prompts, 2, s.n_nodes + 1, s.v_eff), std=0.7)
        st.update(parent=parent, logits=logits, u=mk.uniform((s.n_prompts, s.n_nodes + 1, 2)), out=_outcome(s), q=None, tokens=None)
        if s.n_nodes:
            mixed = logits[:, 1] + s.cfg_scale * (logits[:, 0] - logits[:, 1])
            st["q"], st["tokens"] = _draft(mk, s, parent, near=mixed, noise=4.0)
        return st
    ctx, w = _target(mk, s)
    st.update(ctx=ctx, kv=ctx.kv.view(_dtype(s)))
    if path == "prefill":
        st["prefix"], st["null"] = _prefix(mk, s)
        st["forced"] = mk.ids(s.logit_lo, s.logit_hi, (s.n_prompts, case["forced"])) if case["forced"] else None
        st["u"], st["first"] = mk.uniform((s.n_prompts,)), torch.zeros(s.n_prompts, dtype=torch.int32, device="cuda")
        st["logits"] = torch.empty((s.n_rows, 1, s.v_eff), device="cuda")
        return st
    st["parent"] = parent = _parents(case)
    st["state"] = _start(mk, s, ctx, case["cached"], case.get("ragged", False))
    if path == "step":
        st.update(post=case["post"], out=_outcome(s), logits=torch.empty((s.n_rows, s.n_nodes + 1, s.v_eff), device="cuda"), q=None, tokens=None,
                  u=_clear_uniforms(mk, s, parent, seed, case["post"], case["relaxed"]))
        if s.n_nodes:
            st["q"], st["tokens"] = _draft(mk, s, parent)
        return st
    # a drafter beside the target: four more tokens committed one by one fill the target's feature cache
    out = _outcome(s)
    for _ in range(4):
        ctx.vvs_set_state(st["state"])
        ctx.vvs_verify(0, None, None, None, None, mk.uniform((s.n_prompts, 1, 2)), vb.VVS_STRICT, out["accept_len"], out["path"], out["next"])
        ctx.vvs_kv_commit()
        st["state"][:2] += 1
        st["state"][2] = mk.ids(s.logit_lo, s.logit_hi, (s.n_prompts,))
    own = s.replace(n_layers=1)
    # the drafter proposes from its conditional distribution
    cfg = vb.make_config(own.replace(cfg_scale=1.0), max_nodes=case["context"] + _expanded(parent, s.n_nodes), feature_slots=0, draft_input=1)
    drafter = vb.Context(cfg)
    names = synth.drafter_weight_names()
    dw = _weights(mk, own, [n for n in names if n not in ("embed", "prefix_embed", "wout")])
    dw.update({n: w.get(n) for n in ("embed", "prefix_embed", "wout")})
    drafter.vvs_load_weights([dw[n] for n in names])
    st.update(drafter=drafter, context=case["context"], recent=mk.ids(s.logit_lo, s.logit_hi, (s.n_prompts, case["context"])), given=None,
              tokens=torch.zeros((s.n_prompts, s.n_nodes), dtype=torch.int32, device="cuda"),
              q=torch.zeros((s.n_prompts, s.n_nodes + 1, s.v_eff), device="cuda"))
    if path == "draft":
        st["given"] = _draft(mk, s, parent)[1]
        return st
    st["codebook"] = torch.nn.functional.normalize(mk.normal((s.vocab, 8)), dim=1)
    ctx.vvs_set_codebook(st["codebook"])
    st.update(out=out, u=mk.uniform((s.n_prompts, s.n_nodes + 1, 2)), logits=torch.empty((s.n_rows, s.n_nodes + 1, s.v_eff), device="cuda"))
    return st


# ------------------------------------------------------------------------------------------------ one pass
def _read_logits(ctx, logits):
    status = vb.lib.vvs_debug_logits(ctx.h, logits.data_ptr(), None, None, torch.cuda.current_stream().cuda_stream)
    if status != vb.VVS_OK:
        raise vb.VvsError(status, "vvs_debug_logits")
    return logits


def run(st):
    ctx, path = st["ctx"], st["path"]
    if path == "accept":
        o = st["out"]
        ctx.vvs_accept_from_logits(st["n"], st["parent"], None, st["logits"], st["tokens"], st["q"], st["u"], st["mode"],
                                   o["accept_len"], o["path"], o["next"])
        return o
    if path == "prefill":
        ctx.vvs_prefill(st["prefix"], st["null"], st["forced"], st["u"], st["first"])
        return {"logits": _read_logits(ctx, st["logits"]), "kv": st["kv"]}
    if path == "draft":
        st["drafter"].vvs_draft(ctx, st["n"], st["parent"], None, st["context"], st["recent"], 0, st["given"], st["tokens"], st["q"])
        return {"tokens": st["tokens"], "q": st["q"]}
    o = st["out"]
    ctx.vvs_set_state(st["state"])
    if path == "loop":
        st["drafter"].vvs_draft(ctx, st["n"], st["parent"], None, st["context"], st["recent"], 0, None, st["tokens"], st["q"])
        similarity = ctx.vvs_path_similarity(st["n"], st["parent"], None, st["tokens"], 0.8, 2)
        ctx.vvs_verify(st["n"], st["parent"], None, st["tokens"], st["q"], st["u"], st["mode"], o["accept_len"], o["path"], o["next"])
        logits = _read_logits(ctx, st["logits"])
        ctx.vvs_kv_commit()
        return {"tokens": st["tokens"], "q": st["q"], "similarity": similarity, "logits": logits, "kv": st["kv"], **o}
    if st["post"]:
        ctx.vvs_verify_post(st["n"], st["post"], st["parent"], None, st["tokens"], st["q"], st["u"], st["mode"], o["accept_len"], o["path"], o["next"])
    else:
        ctx.vvs_verify(st["n"], st["parent"], None, st["tokens"], st["q"], st["u"], st["mode"], o["accept_len"], o["path"], o["next"])
    logits = _read_logits(ctx, st["logits"])
    ctx.vvs_kv_commit()
    return {"path": o["path"], "logits": logits, "kv": st["kv"]}
