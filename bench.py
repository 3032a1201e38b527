#!/usr/bin/env python3
"""Benchmark of the per-decode-step vocabulary mask on one MI355X.

A "step" is one pass of the whole hot path over one batch: advance every row by its next token
(host Earley + ZapFormat compaction), compute_mask and apply_mask on that step's logits -- enqueued
with one call, zf_compute_mask_apply_async: the rows' states go up in the kernel's argument block, the
mask kernel over the persistent automaton writes the mask rows in token order, a second launch masks the
logits (a call that meets states for the first time masks up to 16 MB of them in the mask kernel) --
and mask_wait (deferred error check).  The same steps through the two separate calls are reported beside it (`two_calls`).  The token
trajectory is fixed beforehand (tests/golden/trajectory_cfgN.txt, sampled by the CPU oracle), so
nothing is copied back to the host inside the timed region.  Inputs are seeded and synthetic.

Prints ONE JSON line.  `value` = batch * V * steps / wall time of a pass in which every step ends
with the stream synchronised (a decode loop samples step t+1's token from step t's masked logits),
the median of three such passes.  Every pass starts with the rows at the beginning of the trajectory
and the persistent automaton and the state cache cleared (back to what the engine knew when it was
compiled: the states it explored from the empty prefix then, see `without_precomputation`), takes the first `--warmup` steps of the
trajectory untimed and the next `--steps` steps timed: every step of the trajectory is met once per
pass, so nothing a pass has seen before serves its timed steps, beyond what the same rows' earlier
steps have left in the engine.  The same steps without the per-step stream synchronisation are
reported beside it.
"""
import argparse
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# instruction issue peak of the chip: 256 compute units x 4 SIMDs x one wavefront instruction per cycle x 2.4 GHz
ISSUE_PEAK_GINST = 256 * 4 * 2.4
KERNEL_OF_MODE = {0: "mask_automaton_kernel", 1: "mask_walk_kernel", 2: "mask_look_kernel / mask_store_kernel"}

# HBM traffic of one launch of mask_look_kernel (every launch of the default workload is one; masks and logits) and of apply_mask_vec_kernel, from rocprofv3
# FETCH_SIZE / WRITE_SIZE runs scaled by a plain copy of known size (profiles/mask_look_kernel_cfg3_hbm_traffic.txt), and SQ_INSTS of the same
# pass.  The figures describe the kernel sources with the digest below; once they change they are reported as null until measured again.
MEASURED_TRAFFIC = {"config": 3, "bytes_per_launch": 11492183, "apply_bytes_per_launch": 8493664, "instructions_per_launch": 2183682,
                    "kernel_sources_sha256": "61d3ef8574356516efc2403f75cde538786dba1114402c7fcdeb70a3fe5e8ae1"}


def kernel_sources_digest():
    import hashlib
    h = hashlib.sha256()
    for name in ("zf_kernels.hip", "zf_mask_store.hip", "zf_mask_look.hip", "zf_aut_step.h", "zf_mask_automaton.hip", "zf_mask_walk.hip", "zf_kernel_common.h", "zf_launch.h", "zf_device.h",
                 "zf_api.cpp",                                 # the host chooses the launch shape, which decides what the XCDs' L2s share
                 "zf_compile.cpp", "zf_vocab.hip", "zf_host_automaton.h"):   # and how many strings the cache rows leave to a launch
        with open(os.path.join(ROOT, "paper_2506_01151_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def load_trajectory(idx, rows, steps):
    path = os.path.join(ROOT, "tests", "golden", f"trajectory_cfg{idx}.txt")
    if not os.path.exists(path):
        return []
    traj = [[int(x) for x in line.split()] for line in open(path) if line.strip() and not line.startswith("#")]
    if not traj or len(traj[0]) < rows:
        return []
    return [t[:rows] for t in traj[:steps]]


def extend_trajectory(zf, eng, cfg, traj, rows, steps):
    """Continue the trajectory with the library itself (untimed set-up work; the line says so)."""
    import numpy as np
    import torch
    from workloads.configs import pick_set_bit
    from workloads.rng import stream
    states = [eng.new_state() for _ in range(rows)]
    for ids in traj:
        for b, t in enumerate(ids):
            states[b].reset() if t < 0 else states[b].advance(t)
    rs = [stream(cfg.seed, f"bench-extend[{b}]") for b in range(rows)]
    d_mask = torch.empty((rows, eng.W), dtype=torch.int32, device="cuda")
    while len(traj) < steps:
        zf.compute_mask(eng, states, d_mask)
        m = d_mask.cpu().numpy().view(np.uint32)
        ids = []
        for b in range(rows):
            n = int(np.unpackbits(m[b].view(np.uint8)).sum())
            if n == 0:
                states[b].reset()
                ids.append(-1)
            else:
                t = pick_set_bit(m[b], rs[b].below(n))
                states[b].advance(t)
                ids.append(t)
        traj.append(ids)
    return traj


def cpu_baseline(cfg, toks, traj, skip=0, budget_s=15.0):
    """The CPU oracle's mask loop, timed on this host on a bounded sample of (step, row): the timed steps of the
    trajectory (those after the first `skip`), from the first one on, while the budget lasts."""
    from oracle import Oracle
    from workloads import vocab as wvocab
    orc = Oracle(cfg.grammar())
    off, data = wvocab.vocab_csr(toks)
    rows = len(traj[0])
    states = [orc.new_state() for _ in range(rows)]
    n_masks, spent, threads = 0, 0.0, 1
    sample_steps = []
    for step, ids in enumerate(traj):
        for b, t in enumerate(ids):
            if t < 0:
                states[b] = orc.new_state()
            else:
                states[b].feed_bytes(toks[t])
        if step >= skip and spent < budget_s:
            t0 = time.perf_counter()
            for s in states:
                s.mask(off, data, 0)
                n_masks += 1
            spent += time.perf_counter() - t0
            threads = orc.last_threads
            sample_steps.append(step)
    return {"value": n_masks * len(toks) / spent, "unit": "vocab tokens checked/s", "cores": threads, "kind": "oracle",
            "sample": f"{n_masks} masks: all {rows} rows at steps {sample_steps[0] if sample_steps else 0}..{sample_steps[-1] if sample_steps else 0} of the same trajectory (from the first timed step on), {spent:.1f} s"}


def apply_mask_sweep(zf, eng, torch, dtype, batches, launches=24):
    """apply_mask alone at growing batch: each launch works on rows it has not touched for more than
    1.5 GB of traffic (input and output rotate through 3072-row tensors), so nothing is served from
    the last-level cache.  The launches of a shape are recorded into two HIP graphs (a warm-up round and
    the timed round over the next rows), so that the event pair around the timed round spans kernels
    back to back and not the host's launch calls; profiles/ holds the kernel-trace durations of the same sweep."""
    V, W = eng.V, eng.W
    R = 3072
    x = torch.randn((R, V), device="cuda").to(dtype)
    y = torch.empty_like(x)
    m = torch.randint(-2**31, 2**31 - 1, (R, W), dtype=torch.int32, device="cuda")
    esz = x.element_size()
    rows = []
    for B in batches:
        at = 0
        graphs = []
        for _ in range(2):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                for _ in range(launches):
                    zf.apply_mask(eng, x[at:at + B], m[at:at + B], out=y[at:at + B])
                    at = (at + B) % (R - B + 1)
            graphs.append(g)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        graphs[0].replay()
        torch.cuda.synchronize()
        e0.record()
        graphs[1].replay()
        e1.record()
        torch.cuda.synchronize()
        us = e0.elapsed_time(e1) * 1e3 / launches
        nbytes = 2 * B * V * esz + B * W * 4
        rows.append({"batch": B, "us_per_launch": us, "GB/s": nbytes / us / 1e3, "frac": nbytes / us / 1e3 / HBM_PEAK_GBS})
        del graphs
    del x, y, m
    return rows


class Runner:
    """Replays a trajectory through one engine: warm-up steps, then the timed steps from the trajectory's first step."""

    def __init__(self, zf, torch, cfg, eng, traj, logits):
        self.zf, self.torch, self.cfg, self.eng, self.traj, self.logits = zf, torch, cfg, eng, traj, logits
        self.B = len(traj[0])
        self.out = torch.empty_like(logits[0])
        self.d_mask = torch.empty((self.B, eng.W), dtype=torch.int32, device="cuda")
        self.states = zf.StateBatch([eng.new_state() for _ in range(self.B)])

    def run(self, n_warm, n_timed, profile=False, count_hits=False, sync_steps=True, cold=True, keep_masks=None, fused=True):
        zf, torch, eng = self.zf, self.torch, self.eng
        eng.set_profiling(profile)
        lat, adv = [], []
        kern = {"main": [], "finish": [], "apply": []}
        rep = {"overflow": 0, "queued": 0, "steps": 0, "cache_rows": 0, "hits": 0, "upload_bytes": 0}
        evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n_timed)] if profile else None
        stream = torch.cuda.current_stream()
        # the boundary's calls with their arguments marshalled once (the binding's checked wrappers cost a few microseconds a step)
        h_stream = stream.cuda_stream
        p_mask, p_out = self.d_mask.data_ptr(), self.out.data_ptr()
        p_logits = [x.data_ptr() for x in self.logits]
        dt = {torch.float32: 0, torch.bfloat16: 1}[self.out.dtype]
        row_stride = self.out.stride(0)
        t_begin = None
        assert n_warm + n_timed <= len(self.traj), "the trajectory is shorter than warm-up + timed steps"
        for s in self.states:
            s.reset()
        if cold:
            eng.clear_state_cache()                     # a pass starts with nothing: cached masks and the persistent automaton start over
        for i in range(n_warm + n_timed):
            if i == n_warm:     # the timed steps go on where the warm-up steps stopped: every step of the trajectory is met once per pass
                torch.cuda.synchronize()
                t_begin = time.perf_counter()
            k = i - n_warm
            ids = self.traj[i]
            t0 = time.perf_counter()
            self.states.advance(ids)                    # every row by its token (a negative id starts the row over)
            t1 = time.perf_counter()
            if fused:                                   # compute_mask and apply_mask of the step enqueued together by one call
                eng.compute_mask_apply_async(self.states, p_mask, p_logits[i % len(p_logits)], p_out, dt, row_stride, h_stream)
            else:
                eng.compute_mask_async(self.states, p_mask, h_stream)
                if profile and i >= n_warm:
                    evs[k][0].record()
                eng.apply_mask(p_logits[i % len(p_logits)], p_out, dt, self.B, row_stride, p_mask, h_stream)
                if profile and i >= n_warm:
                    evs[k][1].record()
            eng.mask_wait(h_stream)                     # returns once the call's outcome is known; its kernels may still run
            if sync_steps:                              # until the masked logits are there
                stream.synchronize()
            t2 = time.perf_counter()
            if i >= n_warm:
                adv.append(t1 - t0)
                lat.append(t2 - t1)
                if count_hits:
                    rep["hits"] += eng.mask_report().cache_hits
                if profile:
                    r = eng.mask_report()
                    kern["main"].append(r.main_ms)
                    kern["finish"].append(r.permute_ms)
                    rep["overflow"] += r.overflow_chunks
                    rep["queued"] += r.walk_chunks
                    rep["steps"] += r.parser_steps
                    rep["cache_rows"] += r.cache_rows
                    rep["upload_bytes"] += r.chart_bytes
                if keep_masks is not None:
                    keep_masks.append(self.d_mask.clone())
        torch.cuda.synchronize()
        total = time.perf_counter() - t_begin
        if profile and not fused:
            kern["apply"] = [a.elapsed_time(b) for a, b in evs]
        return {"total": total, "lat": lat, "adv": adv, "kern": kern, "rep": rep}


def pct(xs, p):
    return sorted(xs)[min(len(xs) - 1, int(p * len(xs)))]


def side_config(zf, torch, configs, idx, steps, warm, pruning=True, walk_mode=2):
    """A short run of another configuration at its stated batch and vocabulary: synchronised steps, kernel durations
    by HIP events, on the oracle-sampled trajectory."""
    cfg = configs.CONFIGS[idx]
    toks = cfg.vocab()
    traj = load_trajectory(idx, cfg.batch, warm + steps)
    if len(traj) < warm + steps:
        return {"skipped": f"tests/golden/trajectory_cfg{idx}.txt holds {len(traj)} steps of {cfg.batch} rows"}
    eng = zf.Engine(cfg.grammar(), toks, device=0, pruning=pruning, state_cache_entries=-1, walk_mode=walk_mode)
    logits = [configs.make_logits(cfg, i, device="cuda") for i in range(2)]
    rn = Runner(zf, torch, cfg, eng, traj, logits)
    runs = sorted((rn.run(warm, steps, profile=False) for k in range(3)), key=lambda x: x["total"])
    r = runs[1]                                              # three passes, each from a cleared automaton: the median one
    again = rn.run(warm, steps, cold=False) if pruning and walk_mode == 2 else None   # the same steps with the automaton the last pass built
    p = rn.run(warm, steps, profile=True, fused=False)          # two calls: the mask kernel and apply_mask timed separately
    p1 = rn.run(warm, steps, profile=True)                      # one call: the kernel that does both
    B, V = cfg.batch, eng.V
    esz = logits[0].element_size()
    apply_bytes = 2 * B * V * esz + B * eng.W * 4
    apply_ms = statistics.fmean(p["kern"]["apply"])
    out = {"workload": f"configs[{idx - 1}] {cfg.name}: V={V} batch={B} logits={cfg.dtype} pruning={'on' if pruning else 'off'}",
           "trajectory": "oracle-sampled file", "steps": steps, "mask_kernel": KERNEL_OF_MODE[walk_mode] if pruning or walk_mode != 2 else "mask_look_kernel / mask_automaton_kernel",
           "value": B * V * steps / r["total"], "ms_per_step": r["total"] / steps * 1e3, "timed_passes_ms_per_step": [x["total"] / steps * 1e3 for x in runs],
           "p50_mask_apply_latency_us": pct(r["lat"], 0.5) * 1e6, "p99_mask_apply_latency_us": pct(r["lat"], 0.99) * 1e6, "max_mask_apply_latency_us": max(r["lat"]) * 1e6,
           "mean_advance_us_per_step": statistics.fmean(r["adv"]) * 1e6,
           "kernel_ms": {"one_call": statistics.fmean(p1["kern"]["main"]), "two_calls": {k: statistics.fmean(v) for k, v in p["kern"].items() if v}},
           "earley_steps_per_launch": p["rep"]["steps"] / steps, "undecided_strings_per_step": p["rep"]["queued"] / steps,
           "upload_bytes_per_step": p["rep"]["upload_bytes"] / steps,
           "apply_mask": {"algorithmic_bytes": apply_bytes, "GB/s": apply_bytes / (apply_ms * 1e-3) / 1e9, "frac": apply_bytes / (apply_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                          "note": "HIP events around one launch at the configuration's own shape; the buffers are not rotated here, see apply_mask_sweep"}}
    if again:
        out["warm_automaton_ms_per_step"] = again["total"] / steps * 1e3
    del rn, eng
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=480, help="timed steps of a pass; they follow the warm-up steps on the same trajectory (default: 32 + 480 = the 512 oracle-sampled steps)")
    ap.add_argument("--warmup", type=int, default=32, help="untimed steps at the start of every pass")
    ap.add_argument("--config", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-side-configs", action="store_true", help="leave configurations 4 and 5 and the apply_mask sweeps out")
    ap.add_argument("--pruning", type=int, default=1)
    ap.add_argument("--walk-mode", type=int, default=2, help="mask kernel of the headline: 2 = persistent automaton (default), 0 = per-block automaton, 1 = trie walk")
    ap.add_argument("--headline-only", action="store_true",
                    help="run the warm-up and timed steps of one headline pass and nothing else (for hardware-counter runs, "
                         "where every dispatch of a kernel should belong to the same workload); prints a short JSON line")
    ap.add_argument("--traffic-calibration", action="store_true",
                    help="only run apply_mask with an all-ones mask on a [1024, V] tensor three times: a plain copy of known "
                         "size, used to scale rocprofv3's FETCH_SIZE / WRITE_SIZE counters")
    ap.add_argument("--apply-sweep-only", action="store_true", help="only the apply_mask sweeps (for a kernel trace of them)")
    ap.add_argument("--two-calls", action="store_true", help="with --headline-only: the steps through zf_compute_mask_async + zf_apply_mask instead of the one call")
    ap.add_argument("--no-exploration", action="store_true", help="with --headline-only: an engine compiled with precompute_states = -1 (first visits go through mask_store_kernel)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("this benchmark runs on one GPU only: rows and vocabulary ranges would shard without any exchange, "
              "but no multi-GPU path is part of it; run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import paper_2506_01151_amd as zf
    from workloads import configs

    assert torch.cuda.is_available(), "bench.py needs the MI355X"
    cfg = configs.CONFIGS[args.config]
    B, K, Wm = cfg.batch, args.steps, args.warmup
    toks = cfg.vocab()
    # headline engine: state cache off, so every row of every step goes through the mask kernels
    eng = zf.Engine(cfg.grammar(), toks, device=0, pruning=bool(args.pruning), state_cache_entries=-1, walk_mode=args.walk_mode,
                    precompute_states=-1 if args.headline_only and args.no_exploration else 0)
    V, W = eng.V, eng.W
    traj = load_trajectory(args.config, B, Wm + K)
    traj_src = "oracle-sampled file"
    if len(traj) < Wm + K:
        traj_src = f"library-sampled beyond step {len(traj)}, not oracle-checked"
        traj = extend_trajectory(zf, eng, cfg, traj, B, Wm + K)

    if args.traffic_calibration:
        x = torch.zeros((1024, V), dtype=torch.bfloat16, device="cuda")
        y = torch.empty_like(x)
        ones = torch.full((1024, W), -1, dtype=torch.int32, device="cuda")
        for _ in range(3):
            zf.apply_mask(eng, x, ones, out=y)
        torch.cuda.synchronize()
        print(json.dumps({"calibration_copy_bytes_read": x.numel() * 2 + ones.numel() * 4, "calibration_copy_bytes_written": y.numel() * 2}))
        return
    if args.apply_sweep_only:
        print(json.dumps({"bf16": apply_mask_sweep(zf, eng, torch, torch.bfloat16, (16, 64, 256, 1024)),
                          "f32": apply_mask_sweep(zf, eng, torch, torch.float32, (16, 64, 256, 1024))}))
        return

    logits = [configs.make_logits(cfg, i, device="cuda") for i in range(4)]
    esz = logits[0].element_size()
    rn = Runner(zf, torch, cfg, eng, traj, logits)

    if args.headline_only:
        r = rn.run(Wm, K, fused=not args.two_calls)
        print(json.dumps({"headline_only": True, "calls_per_step": "two" if args.two_calls else "one", "steps": K, "warmup": Wm,
                          "ms_per_step": r["total"] / K * 1e3, "value": B * V * K / r["total"]}))
        return

    # three synchronised passes (each from a cleared store): the headline is their median; latencies over all of them
    sync = [rn.run(Wm, K) for k in range(3)]
    sync_totals = sorted(r["total"] for r in sync)
    total = sync_totals[1]
    lat = [x for r in sync for x in r["lat"]]
    adv = [x for r in sync for x in r["adv"]]
    piped = rn.run(Wm, K, sync_steps=False)                       # steps enqueued back to back: the host runs ahead of the stream
    warm = rn.run(Wm, K, cold=False)                              # the same steps again with the persistent automaton left as the last pass built it
    masks = []
    prof = rn.run(Wm, K, profile=True, keep_masks=masks if K <= 1024 else None)   # HIP events around the kernel
    kern, rep = prof["kern"], prof["rep"]
    two = rn.run(Wm, K, fused=False)                              # the same steps through compute_mask_async + apply_mask: two kernels
    two_prof = rn.run(Wm, K, profile=True, fused=False)
    # mask density: allowed fraction per (step, row), from the masks the profiled pass produced
    density_hist = None
    if masks:
        lut = torch.tensor([bin(i).count("1") for i in range(256)], dtype=torch.int32, device="cuda")
        dens = torch.stack([lut[m.view(torch.uint8).long()].sum(dim=1) for m in masks]).float().flatten().cpu().numpy() / V
        edges = [0, 1e-4, 1e-3, 1e-2, 0.05, 0.1, 0.2, 0.4, 0.6, 0.8, 1.0000001]
        counts, _ = np.histogram(dens, bins=edges)
        density_hist = {"allowed_fraction_bin_edges": edges[:-1] + [1.0], "row_steps": [int(c) for c in counts], "mean": float(dens.mean())}
        del masks
    # the same steps with the state cache (Section 5.2) on, starting cold
    eng_sc = zf.Engine(cfg.grammar(), toks, device=0, pruning=bool(args.pruning), walk_mode=args.walk_mode)
    sc = Runner(zf, torch, cfg, eng_sc, traj, logits).run(Wm, K, count_hits=True)
    del eng_sc
    # and with the other mask kernels, state cache off
    others = {}
    for mode in (0, 1, 2):
        if mode == args.walk_mode:
            continue
        eng_alt = zf.Engine(cfg.grammar(), toks, device=0, pruning=bool(args.pruning), state_cache_entries=-1, walk_mode=mode)
        r = Runner(zf, torch, cfg, eng_alt, traj, logits).run(Wm, K)
        others[KERNEL_OF_MODE[mode]] = {"value": B * V * K / r["total"], "ms_per_step": r["total"] / K * 1e3, "p50_mask_apply_latency_us": pct(r["lat"], 0.5) * 1e6}
        del eng_alt

    # the headline pass on an engine compiled without the exploration of the automaton from the empty prefix (zf_options.precompute_states = -1):
    # every pass then starts from a store that knows the empty prefix only
    no_pre = None
    if args.walk_mode == 2 and args.pruning:
        eng_np = zf.Engine(cfg.grammar(), toks, device=0, pruning=True, state_cache_entries=-1, walk_mode=2, precompute_states=-1)
        rn_np = Runner(zf, torch, cfg, eng_np, traj, logits)
        tt = sorted(rn_np.run(Wm, K)["total"] for _ in range(3))
        no_pre = {"ms_per_step": tt[1] / K * 1e3, "value": B * V * K / tt[1],
                  "note": "the same three passes on an engine compiled with precompute_states = -1: a cleared automaton then holds the state of the empty prefix and nothing else"}
        del rn_np, eng_np

    ms_per_step = total / K * 1e3
    value = B * V * K / total
    info = eng.info
    main_ms = statistics.fmean(kern["main"])
    apply_ms = statistics.fmean(two_prof["kern"]["apply"])
    apply_bytes = 2 * B * V * esz + B * W * 4
    # Algorithmic bytes of one launch of the default kernel, once per state that rows of the call stand in: the token-mask-cache words
    # merged (two bitsets of W words per selected cache row), the mask words written, 16 bytes per undecided token (its first fifteen
    # byte classes and a mark), and the upload.  The other mask kernels work in string-rank order (Wr words per row,
    # 24 bytes per undecided string).  The default kernel masks the logits as well: they are read and written.
    Wr = (info.n_strings + 31) // 32
    queued, crows = rep["queued"], rep["cache_rows"]
    if args.walk_mode == 2 and args.pruning:
        mask_bytes = int(crows / K * W * 8 + B * W * 4 + queued / K * 16 + rep["upload_bytes"] / K) + 2 * B * V * esz
    elif args.walk_mode != 1:
        mask_bytes = int(crows / K * Wr * 8 + B * Wr * 4 + queued / K * 24 + rep["upload_bytes"] / K)
    else:
        n_chunks = (info.n_strings + 31) // 32
        mask_bytes = info.n_trie_nodes * 16 + n_chunks * (8 + 64) + B * n_chunks * 4 + int(rep["upload_bytes"] / K)
    traffic_ok = (args.config == MEASURED_TRAFFIC["config"] and args.pruning == 1 and args.walk_mode == 2
                  and kernel_sources_digest() == MEASURED_TRAFFIC["kernel_sources_sha256"])
    kname = KERNEL_OF_MODE[args.walk_mode]
    insts = MEASURED_TRAFFIC["instructions_per_launch"] if traffic_ok else None
    result = {
        "metric": "vocab tokens checked/sec + p50 mask+apply latency per step (V=128k, B=16)",
        "value": value, "unit": "vocab tokens checked/s", "n_gpus": 1, "steps": K, "warmup": Wm,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "u32", "data": "synthetic",
        "config": {"workload": f"configs[{args.config - 1}] {cfg.name}: grammar={cfg.grammar().name} V={V} batch={B} "
                               f"logits={cfg.dtype} pruning={'on' if args.pruning else 'off'}", "trajectory": traj_src,
                   "trajectory_steps": f"steps 0..{Wm - 1} untimed (warm-up), steps {Wm}..{Wm + K - 1} timed, in every pass",
                   "mask_kernel": kname},
        "timed_passes": {"n": 3, "ms_per_step": [t / K * 1e3 for t in sync_totals],
                         "note": "every step ends with the stream synchronised; each pass starts from a persistent automaton cleared back to its compile-time content, runs the warm-up steps and then the timed steps of the same trajectory; value = the median pass"},
        "decode_tokens_per_s": B * K / total,      # one constraint-satisfying token per row and step (the unit of the paper's Table 1)
        "paper_context": "Table 1 of the paper: 8,207.85 tokens/s for its CPU engine on Llama3 / json_schema (parsing + mask generation, "
                         "RTX 3090 + EPYC 7452 host, real tokenizer and data): other hardware, other inputs; context, not a baseline",
        "p50_mask_apply_latency_us": pct(lat, 0.5) * 1e6, "p90_mask_apply_latency_us": pct(lat, 0.9) * 1e6,
        "p99_mask_apply_latency_us": pct(lat, 0.99) * 1e6, "max_mask_apply_latency_us": max(lat) * 1e6,
        "mean_advance_us_per_step": statistics.fmean(adv) * 1e6,
        "pipelined_steps": {"ms_per_step": piped["total"] / K * 1e3, "value": B * V * K / piped["total"],
                            "note": "the same steps without the stream synchronisation: a step ends when zf_mask_wait has returned, which is when the call's outcome is known -- "
                                    "for a call of look-ups, which is not expected to fail, when it is enqueued; the passes' total ends with the stream synchronised, so every kernel is in it: "
                                    "a decode loop whose sampler runs on the same stream"},
        "warm_automaton": {"ms_per_step": warm["total"] / K * 1e3, "value": B * V * K / warm["total"], "p50_mask_apply_latency_us": pct(warm["lat"], 0.5) * 1e6,
                           "note": "the same steps once more without clearing the persistent automaton: every transition is a look-up"},
        "kernel_ms": {k: statistics.fmean(v) for k, v in kern.items() if v},
        "kernel_ms_p50": {k: pct(v, 0.5) for k, v in kern.items() if v},
        "kernel_ms_max": {k: max(v) for k, v in kern.items() if v},
        "two_calls": {"value": B * V * K / two["total"], "ms_per_step": two["total"] / K * 1e3, "p50_mask_apply_latency_us": pct(two["lat"], 0.5) * 1e6,
                      "kernel_ms": {k: statistics.fmean(v) for k, v in two_prof["kern"].items() if v},
                      "note": "the same steps through zf_compute_mask_async + zf_apply_mask: the mask kernel, then apply_mask_vec_kernel (the one call masks the logits in the kernel that works the masks out)"},
        "overflow_chunks_per_step": rep["overflow"] / K,
        ("undecided_tokens_per_step" if args.walk_mode == 2 and args.pruning else "undecided_strings_per_step") if args.walk_mode != 1 else "walk_chunks_per_step": queued / K,
        "undecided_per_s": queued / max(sum(kern["main"]) * 1e-3, 1e-12),
        "earley_steps_per_launch": rep["steps"] / K,
        "token_mask_cache_rows_per_step": crows / K,
        "upload_bytes_per_step": rep["upload_bytes"] / K,
        "mask_density": density_hist,
        "with_state_cache": {"value": B * V * K / sc["total"], "ms_per_step": sc["total"] / K * 1e3,
                             "p50_mask_apply_latency_us": pct(sc["lat"], 0.5) * 1e6, "p99_mask_apply_latency_us": pct(sc["lat"], 0.99) * 1e6,
                             "row_hit_rate": sc["rep"]["hits"] / (B * K),
                             "note": "cache cleared when the timed steps start; the headline value runs with it off"},
        "other_mask_kernels": others,
        "without_precomputation": no_pre,
        "roofline": {"bound": "hbm", "kernel": kname, "achieved": mask_bytes / (main_ms * 1e-3) / 1e9,
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": mask_bytes / (main_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                     "traffic": MEASURED_TRAFFIC["bytes_per_launch"] if traffic_ok else None, "algorithmic_bytes": mask_bytes,
                     "note": "one launch = the mask of every row, worked out once per state that rows stand in, and the rows' logits masked by wavefronts of their own; integer work (a table walk per undecided token), "
                             "bounded by the chain of dependent memory round trips of a wavefront (the group's record, cache words, strings, table "
                             "entries: about 1 us each), far below the HBM roof; the event pair also spans the dispatch gap before the kernel; "
                             "roofline_apply_mask is the logits' masking as a call of its own"},
        "roofline_issue": {"bound": "alu", "kernel": kname, "unit": "G wavefront instructions/s", "peak": ISSUE_PEAK_GINST, "instructions": insts,
                           "achieved": insts / (main_ms * 1e-3) / 1e9 if insts else None,
                           "frac": insts / (main_ms * 1e-3) / 1e9 / ISSUE_PEAK_GINST if insts else None,
                           "note": "instruction count from the SQ_INSTS counter of the profiled run (null once the kernel sources change)"},
        "roofline_apply_mask": {"bound": "hbm", "kernel": "apply_mask_vec_kernel", "achieved": apply_bytes / (apply_ms * 1e-3) / 1e9,
                                "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": apply_bytes / (apply_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                                "traffic": MEASURED_TRAFFIC["apply_bytes_per_launch"] if traffic_ok else None, "algorithmic_bytes": apply_bytes,
                                "note": f"{apply_bytes / 1e6:.1f} MB per launch at this configuration's shape, event pair around one launch; "
                                        "see apply_mask_sweep for the cache-cold sweep over batch sizes"},
    }
    del rn
    if not args.no_side_configs:
        result["apply_mask_sweep"] = {"V": V, "bound": "hbm", "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                      "bf16": apply_mask_sweep(zf, eng, torch, torch.bfloat16, (16, 64, 256, 1024)),
                                      "f32": apply_mask_sweep(zf, eng, torch, torch.float32, (64, 256))}
        result["config_4"] = side_config(zf, torch, configs, 4, 96, 8)
        # from an empty automaton the per-block kernel is the faster one at this shape (the two are level once the automaton has grown)
        result["config_4_per_block_automaton"] = side_config(zf, torch, configs, 4, 96, 8, walk_mode=0)
        result["config_5_pruning_on"] = side_config(zf, torch, configs, 5, 96, 8, pruning=True)
        result["config_5_pruning_off"] = side_config(zf, torch, configs, 5, 96, 8, pruning=False)
    if not args.no_cpu_baseline:
        # the oracle's sample starts with the timed steps and, when those are few, goes on along the same trajectory until its time budget is used
        full = load_trajectory(args.config, B, 1 << 30)
        result["cpu_baseline"] = cpu_baseline(cfg, toks, full if len(full) >= Wm + K and traj_src == "oracle-sampled file" else traj[:Wm + K], skip=Wm)
    print(json.dumps(result))


if __name__ == "__main__":
    main()
