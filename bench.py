#!/usr/bin/env python3
"""Benchmark of the verify pass on one MI355X.

A step = one pass of the whole hot path over one batch: vvs_verify (embedding, L transformer layers
over the T = N + 1 query tokens of every row against the KV cache, lm_head, CFG mix, softmax,
accept / resample, path walk) followed by vvs_kv_commit.  Every step starts from the same saved
per-prompt state (vvs_set_state, one tiny kernel, inside the timed region), so all steps do the same
work at the same cache length.  Inputs are synthetic, seeded, and resident in HBM before timing starts.

Default workload: the LlamaGen-XL shape with a 26-node depth-6 draft tree, 8 prompts x 2 CFG rows,
at mid-image cache length.  Prints one JSON line."""
import argparse
import dataclasses
import json
import re
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X published HBM3E bandwidth
MFMA_BF16_PEAK_TFLOPS = 2500.0   # MI355X published dense bf16 MFMA rate
FP32_VALU_PEAK_TFLOPS = 157.3


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def correlated_draft(synth, shape, parent, noise_std, draft_index, mixed_logits_of):
    """Synthetic drafter of tunable quality.  Level by level: get the target's mixed logits for the current
    draft (mixed_logits_of(q, toks, u) -> [B, T, V_eff]: one verify pass of whoever is asked - the library on
    the GPU, or the checker for its own baseline), let the draft distribution of the nodes of depth k be the
    normalised exponential of (target logits + Gaussian noise), and draw their children from it without
    replacement.  After depth passes every internal node has a draft distribution that resembles the target's,
    as a trained drafter's would.  Not timed."""
    B, N, V = mixed_logits_of.n_prompts, shape.n_nodes, shape.v_eff
    T = N + 1
    depth = synth.node_depths(parent)
    rng = np.random.default_rng(shape.seed + 99 + 7919 * draft_index)
    q = np.full((B, T, V), 1.0 / V, dtype=np.float32)
    toks = rng.integers(shape.logit_lo, shape.logit_hi, size=(B, N)).astype(np.int32)
    u = synth.make_uniforms(shape, N, draft_index)[:B]
    children = {}
    for j in range(1, T):
        children.setdefault(int(parent[j - 1]), []).append(j)
    for level in range(int(depth.max())):
        mixed = mixed_logits_of(q, toks, u)
        for j in [j for j in range(T) if depth[j] == level and j in children]:
            lg = mixed[:, j, :].astype(np.float64) + noise_std * rng.standard_normal((B, V))
            lg -= lg.max(axis=1, keepdims=True)
            e = np.exp(lg)
            qj = e / e.sum(axis=1, keepdims=True)
            q[:, j, :] = qj.astype(np.float32)
            for b in range(B):
                w = q[b, j].astype(np.float64)
                w /= w.sum()
                nz = int((w > 0).sum())
                kids = children[j]
                picks = rng.choice(V, size=len(kids), replace=False, p=w) if nz >= len(kids) else rng.choice(V, size=len(kids), replace=False)
                for c, x in zip(kids, picks):
                    toks[b, c - 1] = shape.logit_lo + int(x)
    return q, toks, u


def build_correlated_draft(ctx, vb, synth, shape, parent, torch, noise_std, bufs, n_post=0, draft_index=0):
    """correlated_draft() with the library's own verify pass as the source of the target logits."""
    dev = ctx.device
    state = bufs["state"]

    def gpu_mixed(q, toks, u):
        ctx.vvs_set_state(state)
        ctx.vvs_verify_post(shape.n_nodes, n_post, parent, None, torch.from_numpy(toks).to(dev), torch.from_numpy(q).to(dev),
                            torch.from_numpy(u).to(dev), vb.VVS_STRICT, bufs["a"], bufs["path"], bufs["next"])
        _, mixed, _ = ctx.vvs_debug_logits()
        return mixed.cpu().numpy()

    gpu_mixed.n_prompts = shape.n_prompts
    out = correlated_draft(synth, shape, parent, noise_std, draft_index, gpu_mixed)
    ctx.vvs_set_state(state)
    return out


def algorithmic_counts(shape, S_mean):
    """Bytes and flops one verify call must move / do (weights once, KV cache once, draft probs once)."""
    L, d, F, V = shape.n_layers, shape.d_model, shape.d_ff, shape.v_eff
    R, T, B = shape.n_rows, shape.n_nodes + 1, shape.n_prompts
    M = R * T
    w_bytes = 2 * (L * (4 * d * d + 3 * d * F) + d * V)
    kv_read = R * L * 2 * S_mean * d * 2
    kv_write = R * L * 2 * T * d * 2
    q_read = B * T * V * 4
    gemm_flops = 2 * M * (L * (4 * d * d + 3 * d * F) + d * V)
    attn_flops = 4 * T * (S_mean + T) * d * L * R
    return dict(w_bytes=w_bytes, kv_read=kv_read, kv_write=kv_write, q_read=q_read, gemm_flops=gemm_flops,
                attn_flops=attn_flops, M=M)


def cpu_baseline(shape, weights, synth, n_forced, u_first, parent, noise_std, mode, nbr, log_fn, n_sample=2, reps=5, n_post=0):
    """The CPU checker as it stands, timed on a bounded sample of the same workload: the first
    n_sample prompts (2 CFG rows each) at the same cache length, with the same tree and a draft of the
    same recipe (draft set 0), built from the checker's OWN target logits - nothing the checker is given
    comes from the GPU library.  The prefill that builds the cache and the passes that build the draft
    are not timed; verify is timed `reps` times (it does not change the cache), commit once."""
    from oracle import vvs_oracle as vo
    try:
        from threadpoolctl import threadpool_info
        threads = max([p.get("num_threads", 1) for p in threadpool_info() if p.get("user_api") == "blas"] or [os.cpu_count()])
    except Exception:
        threads = os.cpu_count()
    n_sample = min(n_sample, shape.n_prompts)
    s1 = shape.replace(n_prompts=n_sample)
    o = vo.Oracle(dataclasses.asdict(s1), weights)
    if nbr is not None:
        o.set_neighbors(nbr)
    pc, pu = synth.make_prefix(shape)
    forced = synth.make_forced_tokens(shape, n_forced) if n_forced > 0 else None
    t0 = time.perf_counter()
    o.prefill(pc[:n_sample], pu, None if forced is None else forced[:n_sample], u_first[:n_sample])
    log_fn(f"cpu baseline: building the cache of the sample took {time.perf_counter() - t0:.1f} s (not counted)")
    t0 = time.perf_counter()

    def cpu_mixed(q_, toks_, u_):
        o.verify(parent, toks_, q_, u_, 0, n_post=n_post)
        return o.mixed_logits

    cpu_mixed.n_prompts = n_sample
    q, toks, u = correlated_draft(synth, s1, parent, noise_std, 0, cpu_mixed)
    log_fn(f"cpu baseline: building the draft from the checker's own logits took {time.perf_counter() - t0:.1f} s (not counted)")
    t0 = time.perf_counter()
    for _ in range(reps):
        a, _, _ = o.verify(parent, toks, q, u, mode, n_post=n_post)
    t_verify = (time.perf_counter() - t0) / reps
    t0 = time.perf_counter()
    o.kv_commit()
    t_commit = time.perf_counter() - t0
    dt = t_verify + t_commit
    emitted = float(a.sum() + len(a))
    return {"value": emitted / dt, "unit": "verified tokens/s", "cores": int(threads), "kind": "oracle",
            "sample": f"{n_sample} of {shape.n_prompts} prompts ({2 * n_sample} CFG rows), same {s1.n_nodes}-node tree, a draft of the same "
                      f"recipe built from the checker's own logits, cache length {s1.prefix_len}+{n_forced}; verify {t_verify:.2f} s (mean of {reps}) + "
                      f"commit {t_commit:.3f} s for {emitted:.0f} emitted / {n_sample * s1.n_nodes} scored draft tokens"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=40)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="llamagen_xl_tree26")
    ap.add_argument("--image-tokens", type=int, default=-1, help="image tokens already emitted (default: half the grid)")
    ap.add_argument("--draft-noise", type=float, default=-1.0,
                    help="std of the noise between draft and target logits behind `value`; default (< 0): calibrated at run time so that "
                         "the tokens emitted per pass are closest to --target-tpf, the paper's own figure for this acceptance mode")
    ap.add_argument("--target-tpf", type=float, default=0.0,
                    help="tokens per target forward to calibrate the synthetic drafter to (default: 1.22 strict - Table 1, EAGLE-2 row - "
                         "and 2.27 relaxed - mean accept length with fresh features, supplementary tables)")
    ap.add_argument("--traffic-summary", default="",
                    help="text summary of rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of THIS build and command (profsum), from which "
                         "roofline.traffic is taken; without it traffic is null")
    ap.add_argument("--mode", choices=["strict", "relaxed"], default="strict")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--latency-calls", type=int, default=100,
                    help="single calls timed with events, warm and with the caches flushed before each (0 = skip)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also launch a plain 256 MiB copy kernel (k_copy_bytes) three times, for scaling hardware traffic counters")
    ap.add_argument("--graph", action="store_true",
                    help="capture one step (set_state, verify, commit) in a HIP graph and time its replays instead of eager launches")
    ap.add_argument("--drafts", type=int, default=6,
                    help="independent synthetic draft sets (tokens, draft distributions, uniforms) cycled through by the steps, so "
                         "that the accept length behind `value` is a mean over drafts x prompts draws and not one draw")
    ap.add_argument("--post", type=int, default=0,
                    help="post verification: this many unverified tokens of a previous verification-free step ride in front of the "
                         "draft tree (vvs_verify_post); 0 = the plain verify pass of the headline workload")
    ap.add_argument("--no-drafter", action="store_true", help="leave out the separate timing of the draft side (vvs_draft)")
    ap.add_argument("--norm-mode", choices=["auto", "separate"], default="auto",
                    help="vvs_config.norm_mode: separate = always the normalisation kernels that round where the definition does")
    ap.add_argument("--layers", type=int, default=0, help="override depth (debugging only; the result is then not the named workload)")
    ap.add_argument("--prompts", type=int, default=0, help="override the number of prompts (debugging only; the result is then not the named workload)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on ONE GPU; prompts shard across GPUs without any collective, which is not "
              "exercised here.  Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2511_13587_amd import binding as vb
    from paper_2511_13587_amd import synth

    shape = synth.SHAPES[args.workload]
    if args.layers:
        shape = shape.replace(n_layers=args.layers)
    if args.prompts:
        shape = shape.replace(n_prompts=args.prompts)
    if args.post:
        shape = shape.replace(n_nodes=shape.n_nodes + args.post)
    n_emitted = shape.grid // 2 if args.image_tokens < 0 else args.image_tokens
    n_forced = n_emitted - 1
    T_call = shape.n_nodes + 1
    # the cache is prefilled up to the last length a full call still fits in (end of image); the timed states
    # (start / middle / end of the image) are roll-backs of it with vvs_set_state: their K/V are all real forward outputs
    n_forced_end = max(n_forced, shape.grid - T_call - 1)
    mode = vb.VVS_RELAXED if args.mode == "relaxed" else vb.VVS_STRICT

    t0 = time.perf_counter()
    weights = synth.make_weights(shape)
    log(f"weights generated in {time.perf_counter() - t0:.1f} s")
    ctx = vb.Context(vb.make_config(shape, norm_mode=vb.VVS_NORM_SEPARATE if args.norm_mode == "separate" else vb.VVS_NORM_AUTO))
    ctx.load_weights_from_host(weights, synth.weight_names(shape))
    dev = ctx.device
    if shape.relax_k:
        nbr = torch.from_numpy(synth.make_codebook_neighbours(shape.vocab, shape.relax_k)).to(dev)
        ctx.vvs_set_neighbors(nbr)
    log(f"context: kv {ctx.kv_bytes / 2**30:.2f} GiB, workspace {ctx.ws_bytes / 2**30:.2f} GiB, weights {ctx.pw_bytes / 2**30:.2f} GiB")

    B = shape.n_prompts
    pc, pu = synth.make_prefix(shape)
    if shape.prefix_kind == synth.PREFIX_CLASS:
        dpc, dpu = torch.from_numpy(pc).to(dev), None
    else:
        dpc, dpu = vb.to_device(pc, shape.dtype), vb.to_device(pu, shape.dtype)
    forced_host = synth.make_forced_tokens(shape, n_forced_end)
    forced = torch.from_numpy(forced_host).to(dev) if n_forced_end > 0 else None
    first = torch.zeros(B, dtype=torch.int32, device=dev)
    u0_host = np.random.default_rng(1).random(B, dtype=np.float32)
    u0 = torch.from_numpy(u0_host).to(dev)
    t0 = time.perf_counter()
    ctx.vvs_prefill(dpc, dpu, forced, u0, first)
    torch.cuda.synchronize()
    log(f"prefill to cache length {shape.prefix_len}+{n_forced_end}: {time.perf_counter() - t0:.3f} s")
    state_end = ctx.vvs_read_state()

    def rolled_back(nf):
        """state after nf teacher-forced image tokens: cached length P + nf, nf + 1 emitted, pending = forced token nf (or the sampled one)"""
        st = state_end.copy()
        st[0, :] = shape.prefix_len + nf
        st[1, :] = nf + 1
        if nf < n_forced_end:
            st[2, :] = forced_host[:, nf]
        return st

    states = {"start": rolled_back(0), "middle": rolled_back(n_forced), "end": rolled_back(n_forced_end)}
    state0 = states["middle"]
    state = torch.from_numpy(state0).to(dev)
    ctx.vvs_set_state(state)
    bufs = dict(state=state, a=torch.zeros(B, dtype=torch.int32, device=dev),
                path=torch.zeros((B, vb.VVS_MAX_T), dtype=torch.int32, device=dev),
                next=torch.zeros(B, dtype=torch.int32, device=dev))
    parent = synth.tree_parents(shape.tree_widths, shape.n_nodes - args.post)
    if args.post:                                   # the draft tree hangs below a chain of unverified tokens
        parent = np.array(list(range(args.post)) + [int(p) + args.post for p in parent], dtype=np.int32)
    mask = synth.ancestor_mask(parent)
    N = shape.n_nodes

    def build_drafts(noise, n_sets, first_index=0):
        out_ = []
        for di in range(n_sets):
            q_i, toks_i, u_i = build_correlated_draft(ctx, vb, synth, shape, parent, torch, noise, bufs, args.post, first_index + di)
            out_.append((torch.from_numpy(q_i).to(dev), torch.from_numpy(toks_i).to(dev), torch.from_numpy(u_i).to(dev)))
        return out_

    def accept_lengths(sets):
        """accept lengths of every prompt for every draft set, one untimed pass per set from the middle state"""
        acc = []
        for dq_, dtoks_, du_ in sets:
            ctx.vvs_set_state(state)
            ctx.vvs_verify_post(N, args.post, parent, mask, dtoks_, dq_, du_, mode, bufs["a"], bufs["path"], bufs["next"])
            acc.append(bufs["a"].cpu().numpy().copy())
        ctx.vvs_set_state(state)
        return np.concatenate(acc)

    # The synthetic drafter's quality is one knob (noise between its logits and the target's).  `value` uses the
    # setting whose tokens per target forward are closest to what the paper reports for this acceptance mode
    # (Table 1: 1.22 for strict tree verification; supplementary tables: 2.27 with relaxed acceptance); the
    # low-noise setting of earlier runs is reported beside it.
    target_tpf = args.target_tpf if args.target_tpf > 0 else (2.27 if args.mode == "relaxed" else 1.22)
    calibration = None
    noise = args.draft_noise
    if noise < 0:
        calibration = {}
        for cand in (1.0, 2.0, 3.0, 4.0, 5.0, 6.0, 8.0):
            calibration[cand] = float(accept_lengths(build_drafts(cand, 1, first_index=100)).mean() + 1.0)
        noise = min(calibration, key=lambda c: abs(calibration[c] - target_tpf))
        log("draft noise calibration (noise std -> tokens per forward):", calibration, "-> using", noise)
    drafts = build_drafts(noise, max(1, args.drafts))
    drafts_low_noise = build_drafts(1.0, max(1, args.drafts)) if noise != 1.0 else drafts
    dq, dtoks, du = drafts[0]
    counter = [0]

    def step():
        dq_, dtoks_, du_ = drafts[counter[0] % len(drafts)]
        counter[0] += 1
        ctx.vvs_set_state(state)
        ctx.vvs_verify_post(N, args.post, parent, mask, dtoks_, dq_, du_, mode, bufs["a"], bufs["path"], bufs["next"])
        ctx.vvs_kv_commit()

    if args.calibrate_copy:
        src = torch.ones(64 << 20, dtype=torch.float32, device=dev)      # 256 MiB
        dst = torch.empty_like(src)
        for _ in range(3):
            ctx.vvs_debug_copy(dst, src)
        torch.cuda.synchronize()
        del src, dst
    run = step
    if args.graph:
        # the library makes no allocation, copy or memset in these calls, so a step is one capturable chain of kernels
        for _ in range(2):
            step()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        run = graph.replay
    for _ in range(args.warmup):
        run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        run()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = elapsed / args.steps * 1e3
    # accept lengths: every draft set replayed once more (the kernels are deterministic), outside the timed region
    n_sets = 1 if args.graph else len(drafts)               # a captured graph replays draft set 0 only
    accept = accept_lengths(drafts[:n_sets])
    emitted = float(accept.sum() + len(accept)) / n_sets    # mean emitted tokens per step
    value = emitted / (ms_per_step * 1e-3)
    accept_low = accept_lengths(drafts_low_noise[:n_sets])
    hist = np.bincount(accept, minlength=int(synth.node_depths(parent).max()) + 1)
    # the same step at the start and at the end of the image (cache lengths P and P + G - T - 1), same drafts
    latency_by_cache = {}
    for where in ("start", "middle", "end"):
        if where == "middle":
            latency_by_cache[where] = {"cache_len": int(states[where][0, 0]), "ms_per_step": ms_per_step}
            continue
        if args.graph:                                     # a captured graph has the middle state baked in
            continue
        state_mid = state
        state = torch.from_numpy(states[where]).to(dev)
        for _ in range(args.warmup):
            step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            step()
        torch.cuda.synchronize()
        latency_by_cache[where] = {"cache_len": int(states[where][0, 0]), "ms_per_step": (time.perf_counter() - t0) / args.steps * 1e3}
        state = state_mid
    ctx.vvs_set_state(state)

    # latency of single calls (set state + verify + commit), each bracketed by two events on the stream the library
    # launches on: warm = back to back; cold = a 768 MiB fill before every call, which replaces the contents of the
    # 8 x 4 MB L2 and of the 256 MB memory-side cache
    per_call = None
    if not args.graph and args.latency_calls > 0:
        def timed_calls(n, flush):
            ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n)]
            for i, (e0, e1) in enumerate(ev):
                if flush is not None:
                    flush.fill_(float(i))
                e0.record()
                step()
                e1.record()
            torch.cuda.synchronize()
            return np.array([e0.elapsed_time(e1) for e0, e1 in ev])
        warm_t = timed_calls(args.latency_calls, None)
        flush = torch.empty(192 << 20, dtype=torch.float32, device=dev)
        cold_t = timed_calls(args.latency_calls, flush)
        del flush
        per_call = {"calls": args.latency_calls, "cache_len": int(state0[0, 0]),
                    "warm_ms": {"median": float(np.median(warm_t)), "p10": float(np.percentile(warm_t, 10)), "p90": float(np.percentile(warm_t, 90))},
                    "cold_ms": {"median": float(np.median(cold_t)), "p10": float(np.percentile(cold_t, 10)), "p90": float(np.percentile(cold_t, 90))}}
        ctx.vvs_set_state(state)

    # per-kernel-class durations from HIP events recorded by the library on this stream
    ctx.vvs_timing_enable(True)
    tsteps = min(args.steps, 10)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(tsteps):
        step()
    torch.cuda.synchronize()
    event_pass_ms = (time.perf_counter() - t0) / tsteps * 1e3   # this pass is slower than the timed one: two event records per launch
    names = ["gemm", "attention", "accept", "elementwise", "commit"]
    classes = {}
    for k, nm in enumerate(names):
        n, ms = ctx.vvs_timing_read(k)
        classes[nm] = {"launches_per_step": n / tsteps, "ms_per_step": ms / tsteps}
    ctx.vvs_timing_enable(False)
    S_mean = float(state0[0].mean())
    cnt = algorithmic_counts(shape, S_mean)
    one_launch = classes["gemm"]["launches_per_step"] == 2       # all layers, and the output head
    norms = "normalisation in the projections" if ctx.vvs_plan_is_fused(N + 1) else "separate normalisations"
    if one_launch:
        layer_plan = f"all layers in one launch ({norms})"
    elif not ctx.vvs_plan_is_fused(N + 1):
        layer_plan = "separate normalisation kernels (7 launches per layer)"
    elif classes["attention"]["launches_per_step"] == 0:
        layer_plan = "fused (4 launches per layer: projection + attention in one)"
    else:
        layer_plan = "fused (5 launches per layer)"
    dom = max(("gemm", "attention"), key=lambda k: classes[k]["ms_per_step"])
    if dom == "gemm":
        n_launch = classes["gemm"]["launches_per_step"]
        t_launch = classes["gemm"]["ms_per_step"] * 1e-3 / n_launch
        bytes_launch, flops_launch = cnt["w_bytes"] / n_launch, cnt["gemm_flops"] / n_launch
        kernel = "k_gemm_direct + k_gemm_shared_dma (all bf16 projection GEMMs of one verify call)"
        if classes["attention"]["launches_per_step"] == 0:
            # the q/k/v projection and attention, or all layers, run in one launch: its cache traffic and flops belong to these launches
            bytes_launch += (cnt["kv_read"] + cnt["kv_write"]) / n_launch
            flops_launch += cnt["attn_flops"] / n_launch
            kernel = "k_qkv_attn + k_gemm_direct + k_gemm_shared_dma (all projection launches of one verify call; attention runs inside the first)"
        if one_launch:
            kernel = ("k_layers_few" if ctx.vvs_plan_is_fused(N + 1) else "k_layers_wide") + " + the output head (all launches of one verify call that hold projections)"
    else:
        n_launch = classes["attention"]["launches_per_step"]
        t_launch = classes["attention"]["ms_per_step"] * 1e-3 / n_launch
        bytes_launch = (cnt["kv_read"] + cnt["kv_write"]) / n_launch
        flops_launch = cnt["attn_flops"] / n_launch
        kernel = "k_attn_mfma"
    ideal_hbm, ideal_mfma = bytes_launch / (HBM_PEAK_GBS * 1e9), flops_launch / (MFMA_BF16_PEAK_TFLOPS * 1e12)
    if ideal_mfma > ideal_hbm:
        ach = flops_launch / t_launch / 1e12
        roof = {"bound": "mfma", "achieved": ach, "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s", "frac": ach / MFMA_BF16_PEAK_TFLOPS}
    else:
        ach = bytes_launch / t_launch / 1e9
        roof = {"bound": "hbm", "achieved": ach, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": ach / HBM_PEAK_GBS}
    traffic, traffic_source = None, None
    if args.traffic_summary and dom == "gemm":
        # HBM bytes per launch from a summary of rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this build and command,
        # scaled by the same counters' reading for a plain copy kernel (its last line)
        m = re.search(r"HBM traffic per launch \(fetch \+ write\): ([0-9.]+) MB", open(args.traffic_summary).read())
        traffic = float(m.group(1)) * 1e6 if m else None
        traffic_source = os.path.basename(args.traffic_summary)
    roof.update(traffic=traffic, traffic_source=traffic_source, kernel=kernel, launches_per_step=n_launch, avg_launch_us=t_launch * 1e6,
                algorithmic_bytes_per_launch=bytes_launch, algorithmic_flops_per_launch=flops_launch)
    total_bytes = cnt["w_bytes"] + cnt["kv_read"] + cnt["kv_write"] + cnt["q_read"]

    out = {
        "metric": "verified tokens/s + verify latency at XL shape; % HBM/MFMA roofline",
        "value": value, "unit": "verified tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16" if shape.dtype == synth.DTYPE_BF16 else "f32", "data": "synthetic",
        "config": {"workload": shape.name, "prompts": B, "rows": shape.n_rows, "draft_nodes": N, "tree_depth": int(synth.node_depths(parent).max()),
                   "cache_len_mean": S_mean, "mode": args.mode, "draft_noise_std": noise,
                   "draft_noise_calibrated_to_tokens_per_forward": target_tpf if calibration is not None else None,
                   "launch": "hip graph replay" if args.graph else "eager", "post_verified_tokens": args.post,
                   "draft_sets": n_sets, "layer_plan": layer_plan},
        "shape": {"layers": shape.n_layers, "d_model": shape.d_model, "heads": shape.n_heads, "d_ff": shape.d_ff,
                  "allowed_ids": shape.v_eff, "grid": [shape.grid_h, shape.grid_w], "prefix_len": shape.prefix_len},
        "verify_latency_ms": ms_per_step, "mean_accept_len": float(accept.mean()),
        "tokens_per_forward": float(accept.mean()) + 1.0, "accept_len_histogram": [int(v) for v in hist],
        "emitted_tokens_per_step": emitted,
        "draft_noise_calibration": None if calibration is None else {str(k): v for k, v in calibration.items()},
        "at_draft_noise_1.0": {"tokens_per_forward": float(accept_low.mean()) + 1.0,
                               "verified_tokens_per_s": float(accept_low.sum() + len(accept_low)) / n_sets / (ms_per_step * 1e-3)},
        "latency_by_cache_len": latency_by_cache, "latency_per_call": per_call, "caches": "warm (no flush between steps; the weights alone exceed every cache)", "scored_draft_tokens_per_s": B * N / (ms_per_step * 1e-3),
        "whole_pass": {"algorithmic_GB": total_bytes / 1e9, "algorithmic_TFLOP": (cnt["gemm_flops"] + cnt["attn_flops"]) / 1e12,
                       "hbm_frac": total_bytes / (ms_per_step * 1e-3) / (HBM_PEAK_GBS * 1e9),
                       "mfma_frac": (cnt["gemm_flops"] + cnt["attn_flops"]) / (ms_per_step * 1e-3) / (MFMA_BF16_PEAK_TFLOPS * 1e12)},
        "kernel_classes": classes, "kernel_classes_pass_ms_per_step": event_pass_ms,
        "roofline": roof,
    }
    # the dynamic schedule's decision kernel (Eq. 2 on the same draft tree), timed on its own: it is not part of a verify step
    emb = torch.from_numpy(synth.make_codebook_embeddings(shape.vocab)).to(dev)
    ctx.vvs_set_codebook(emb)
    for _ in range(5):
        ctx.vvs_path_similarity(N, parent, None, dtoks, 0.8, 2)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(200):
        sim = ctx.vvs_path_similarity(N, parent, None, dtoks, 0.8, 2)
    torch.cuda.synchronize()
    out["scheduler"] = {"path_similarity_us_per_call": (time.perf_counter() - t0) / 200 * 1e6, "alpha": 0.8, "stride": 2,
                        "mean_similarity": float(sim.mean().item())}
    # the draft side (a one-block drafter of the same width with random weights, five cached features as context,
    # the same tree shape, greedy top-k children), timed on its own: a second workload, not part of `value`
    if not args.no_drafter:
        tree = synth.tree_parents(shape.tree_widths, shape.n_nodes - args.post)
        n_expanded = len(set(int(p_) for p_ in tree if p_ > 0))
        n_ctx = min(5, ctx.cfg.feature_slots)
        dshape = shape.replace(n_layers=1)
        dctx = vb.Context(vb.make_config(dshape, max_nodes=n_ctx + n_expanded - 1, feature_slots=0, draft_input=1))
        dctx.load_weights_from_host(synth.make_drafter_weights(shape, weights), synth.drafter_weight_names())
        recent = torch.from_numpy(np.random.default_rng(3).integers(shape.logit_lo, shape.logit_hi, (B, n_ctx)).astype(np.int32)).to(dev)
        d_tok = torch.zeros((B, len(tree)), dtype=torch.int32, device=dev)
        d_q = torch.zeros((B, len(tree) + 1, shape.v_eff), dtype=torch.float32, device=dev)
        for _ in range(3):
            dctx.vvs_draft(ctx, len(tree), tree, None, n_ctx, recent, 0, None, d_tok, d_q)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(30):
            dctx.vvs_draft(ctx, len(tree), tree, None, n_ctx, recent, 0, None, d_tok, d_q)
        torch.cuda.synchronize()
        out["drafter"] = {"ms_per_call": (time.perf_counter() - t0) / 30 * 1e3, "blocks": 1, "context_pairs": n_ctx,
                          "tree_nodes": len(tree), "levels": int(synth.node_depths(tree).max()), "expanded_nodes": n_expanded + 1,
                          "weights": "random"}
        dctx.close()
        del dctx
    ctx.close()
    del ctx
    if not args.no_cpu_baseline:
        try:
            nbr_host = synth.make_codebook_neighbours(shape.vocab, shape.relax_k) if shape.relax_k else None
            out["cpu_baseline"] = cpu_baseline(shape, weights, synth, n_forced, u0_host, parent, noise, mode, nbr_host, log, n_post=args.post)
        except MemoryError as e:           # pragma: no cover
            out["cpu_baseline"] = {"value": None, "unit": "verified tokens/s", "cores": os.cpu_count(), "kind": "oracle",
                                   "sample": f"failed: {e}"}
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
