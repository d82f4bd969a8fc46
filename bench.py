#!/usr/bin/env python3
"""Benchmark: verify + draft decode attention on one MI355X.

A step is one verification call (gamma+1 speculated tokens of every sequence
against the full cache) plus one draft call (the same queries against the
StreamingLLM-style sink + window cache), i.e. the two attention calls of the
paper's self-speculative decoding at one layer.  The workload is the
Llama-3.1-8B layer shape at B = 64, S = 32768 in a 16-token paged cache,
gamma = 4, draft budget 16 sinks + 1008 window; inputs are seeded synthetic
N(0, 1) values already resident in HBM.

Timing: 80 untimed verify calls (~100 ms: the clocks settle after the
host-side setup), W untimed warm-up steps, then exactly K steps between two
synchronisations.  Inside each step the caches are evicted before each call
by reading a 1 GiB buffer with cache-allocating loads (cold cache; a fill
would leave dirty lines whose write-back the timed call pays for -- both are
reported), and HIP events on the launch stream bracket each call;
ms_per_step and `value` come from those events (eviction excluded), the wall
time of the K-step region is reported beside them.

`value` is K/V HBM GB/s: the algorithmic K/V bytes of verify + draft (every
visible K and V element once) divided by the step time.  `roofline` is for
the dominant kernel (the verify attention kernel, a single launch here):
`achieved`/`frac` from the event times of the K timed calls, and
`kernel_time` from the rocprofv3 kernel trace of the same K timed dispatches
(profiles/, written by this script's --summarize mode from a traced run of
itself); HBM traffic and MFMA utilisation come from the committed rocprofv3
counter summaries.  Each profile is used only while the kernel sources it
was taken on are unchanged (their SHA-256 is recorded in it).  `cpu_baseline`
is the fp64 oracle timed on a bounded sample of the same workload on this
host's cores (a reported baseline, not a target).  `inputs_sha256` identifies
the seeded inputs that were timed.  `detail` adds every configuration of the
workload list (verify, draft, one-token draft and verify, t_SD, GB/s), the
one-token and warm timings, the listed and gathered SnapKV-style drafts, the
SnapKV selection, append, acceptance and commit, whole engine-shaped
speculative steps (eager and as a HIP graph), the read ceiling and the oracle
beside the step kernels.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline]
                       [--no-configs]
       python bench.py --summarize trace|counters|mfma|... --csv F [F2] --bench-json J [J2]
                       --cmd "..."   (writes a profiles/ summary to stdout)
"""
import argparse
import csv
import hashlib
import json
import math
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

WORKLOAD = "llama8b_b64_s32k_paged"
HBM_PEAK_GBS = 8000.0
SETTLE_CALLS = 80  # untimed verify calls before the warm-up steps (see settle())
MFMA_BF16_PEAK_TFLOPS = 2500.0
PROFILES = os.path.join(ROOT, "profiles")
PROFILE_TRACE = os.path.join(PROFILES, "attn_verify_llama8b_b64_s32k_paged_trace.md")
PROFILE_COUNTERS = os.path.join(PROFILES, "attn_verify_llama8b_b64_s32k_paged_counters.md")
PROFILE_MFMA = os.path.join(PROFILES, "attn_mfma_llama8b_b64_s32k_paged.md")
CSRC = os.path.join(ROOT, "paper_2408_11049_amd", "csrc")
# What decides the attention launches' code and plans: their sources, and the
# per-file compiler flags.
KERNEL_SOURCES = [os.path.join(CSRC, f) for f in
                  ("attn_kernel.h", "attn.hip", "attn_agpr.hip", "merge.hip", "api.cpp", "plan.cpp",
                   "internal.h", "kernels.h")]
KERNEL_SOURCES.append(os.path.join(ROOT, "paper_2408_11049_amd", "build.py"))
# Per-config table: the workload list's configurations (the bench workload is
# the headline itself).
CONFIGS = ["tiny_f32", "llama8b_b32_s8k", "llama8b_b64_ragged_paged", "llama8b_b256_s8k_koutlier",
           "llama70b_b16_s128k"]


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_source_sha256(paths=None):
    """SHA-256 over the attention launch's sources (name and bytes of each)."""
    h = hashlib.sha256()
    for path in paths or KERNEL_SOURCES:
        h.update(os.path.basename(path).encode() + b"\0")
        h.update(open(path, "rb").read())
    return h.hexdigest()


def kv_bytes(w, lens, mode, q_len):
    """Algorithmic K+V bytes of one call: every visible element read once.
    Verify: S_b tokens per (sequence, kv head).  Draft: the union over the
    q_len rows of sinks and windows, [0, n_sink) u [S_b - q_len - W + 1, S_b)."""
    per_tok = 2 * w.Hkv * w.d * w.esize
    total = 0
    for S in lens:
        S = int(S)
        if mode == "verify":
            n = S
        else:
            lo = max(0, S - q_len - w.window + 1)
            n = S if lo <= w.n_sink else w.n_sink + (S - lo)
        total += n * per_tok
    return total


def _profile_fields(path):
    """The `key: value` lines of a committed profile summary, or None when it
    is missing or was taken on other kernel sources."""
    if not os.path.exists(path):
        return None
    fields = dict(re.findall(r"^([a-z0-9_]+):\s*(\S+)\s*$", open(path).read(), re.M))
    if fields.get("kernel_source_sha256") != kernel_source_sha256():
        return None
    return fields


def read_counters():
    """HBM bytes (FETCH + WRITE, calibrated) per verify launch, from the
    committed counter summary; None if absent or stale."""
    f = _profile_fields(PROFILE_COUNTERS)
    if not f or "verify_fetch_bytes_per_launch" not in f:
        return None
    return float(f["verify_fetch_bytes_per_launch"]) + float(f["verify_write_bytes_per_launch"])


def read_mfma():
    """The verify kernel's bf16 MFMA rate from the committed counter summary
    (FLOP per launch from SQ_INSTS_VALU_MFMA_MOPS_BF16 over the dispatch's
    duration), or None if absent or stale."""
    f = _profile_fields(PROFILE_MFMA)
    if not f or "verify_mfma_tflops" not in f:
        return None
    t = float(f["verify_mfma_tflops"])
    return {"bf16_tflops": t, "peak_tflops": MFMA_BF16_PEAK_TFLOPS,
            "frac": round(t / MFMA_BF16_PEAK_TFLOPS, 4),
            "busy_pct": float(f["verify_mfma_busy_pct"]) if "verify_mfma_busy_pct" in f else None,
            "source": os.path.relpath(PROFILE_MFMA, ROOT)}


def read_trace():
    """Kernel durations of the timed verify and draft dispatches from the
    committed kernel-trace summary, or None if absent or stale."""
    f = _profile_fields(PROFILE_TRACE)
    if not f or "verify_kernel_mean_us" not in f:
        return None
    return {k: float(v) for k, v in f.items()
            if k.endswith("_us") or k.endswith("_frac") or k.endswith("_bytes")}


# ---------------------------------------------------------------------------
# Profile summaries (--summarize): turn a rocprofv3 run of this script into the
# markdown under profiles/.  The attention dispatches of a run come in a fixed
# order -- the settling verify calls (their count is in the bench line), W
# warm-up steps, then the K timed steps, each a verify call then a draft call
# -- so the timed calls are picked by ordinal, not by guesswork.

def _rows(path):
    with open(path, newline="") as f:
        return list(csv.DictReader(f))


def _short(name):
    name = name.split("(")[0].replace("void ", "")
    return name.strip()


def _dispatches(rows):
    """{dispatch id: {"name", "start", "end", counter: value ...}} in launch order."""
    out = {}
    for r in rows:
        d = int(r["Dispatch_Id"])
        e = out.setdefault(d, {"name": r["Kernel_Name"]})
        if "Start_Timestamp" in r and r.get("Start_Timestamp"):
            e["start"], e["end"] = int(r["Start_Timestamp"]), int(r["End_Timestamp"])
        if "Counter_Name" in r:
            e[r["Counter_Name"]] = e.get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
    return [out[k] for k in sorted(out)]


def settle_count(rec):
    """The untimed verify calls a bench line says ran before its warm-up."""
    for k, v in rec.get("detail", {}).items():
        if k.startswith("settle_calls"):
            return int(v)
    return 0


def attention_calls(dispatches):
    """The run's attention calls in launch order: each an attention dispatch
    plus the merge dispatch that follows it, if any (split plans)."""
    calls, cur = [], None
    for d in dispatches:
        if "attn_partial_kernel" in d["name"]:
            cur = [d]
            calls.append(cur)
        elif ("merge_lse_kernel" in d["name"] or "merge_many_kernel" in d["name"]) and cur is not None:
            cur.append(d)
            cur = None
        else:
            cur = None
    return calls


def timed_calls(dispatches, warmup, steps, settle=0):
    """The timed verify and draft calls: lists of dispatch groups (an
    attention dispatch plus a merge dispatch that follows it, if any), after
    `settle` untimed verify calls and `warmup` warm-up steps."""
    calls = attention_calls(dispatches)
    need = settle + 2 * (warmup + steps)
    if len(calls) < need:
        raise SystemExit(f"only {len(calls)} attention calls; expected at least {need}")
    timed = calls[settle + 2 * warmup: need]
    return timed[0::2], timed[1::2]


def _bench_line(path):
    for line in open(path):
        line = line.strip()
        if line.startswith("{") and '"metric"' in line:
            return json.loads(line)
    raise SystemExit(f"no bench line in {path}")


def summarize_trace(csv_path, bench_json, cmd):
    rec = _bench_line(bench_json)
    W, K, S0 = rec["warmup"], rec["steps"], settle_count(rec)
    ver, dra = timed_calls(_dispatches(_rows(csv_path)), W, K, S0)
    det = rec["detail"]
    ev = {"verify": det["t_verify_us"], "draft": det["t_draft_us"]}
    alg = {"verify": det["verify_kv_bytes"], "draft": det["draft_kv_bytes"]}
    out = ["# Kernel timing of the bench's timed verify and draft calls (rocprofv3 kernel trace)",
           "",
           f"Workload: {WORKLOAD} -- Llama-3.1-8B layer shape, B = 64, S = 32768, 16-token pages,",
           "gamma = 4, draft 16 sinks + 1008 window, bf16; cold cache (a 1 GiB read evicts the",
           "caches before every call).  One MI355X (gfx950).",
           "",
           "Command (from /tmp with TMPDIR=/tmp; R = the repository root); its stdout is the",
           "bench line quoted below:",
           "",
           f"    {cmd}",
           "",
           f"Selection: bench.py runs {S0} untimed verify calls (settling the clocks), then",
           f"W = {W} warm-up steps and K = {K} timed steps, each a verify call followed by a",
           "draft call, before any other attention call, so in launch order the attention",
           "dispatches go verify x settle, then verify, draft, verify, draft, ...  The",
           f"timed verify calls are attention dispatches {S0 + 2 * W}, {S0 + 2 * W + 2}, ..., "
           f"{S0 + 2 * (W + K) - 2} (0-based), the",
           f"timed draft calls {S0 + 2 * W + 1}, ..., {S0 + 2 * (W + K) - 1}; a merge dispatch that "
           "follows a call",
           "(split plans only) counts with it.",
           "",
           "| call | kernel | timed calls | kernel mean us | min | max | event mean us (bench line) | kernel / event | K/V GB/s (kernel) | frac of 8 TB/s (kernel) | frac (event) |",
           "|---|---|---|---|---|---|---|---|---|---|---|"]
    fields = {"kernel_source_sha256": kernel_source_sha256(), "settle": S0, "warmup": W,
              "steps": K}
    for name, calls in (("verify", ver), ("draft", dra)):
        durs = [sum((d["end"] - d["start"]) for d in c) / 1e3 for c in calls]
        kn = sorted({_short(d["name"]) for c in calls for d in c})
        mean = sum(durs) / len(durs)
        gbs = alg[name] / (mean * 1e-6) / 1e9
        out.append(f"| {name} | {' + '.join('`%s`' % k for k in kn)} | {len(durs)} | {mean:.2f} | "
                   f"{min(durs):.2f} | {max(durs):.2f} | {ev[name]:.2f} | {mean / ev[name]:.4f} | "
                   f"{gbs:.1f} | {gbs / HBM_PEAK_GBS:.4f} | "
                   f"{alg[name] / (ev[name] * 1e-6) / 1e9 / HBM_PEAK_GBS:.4f} |")
        fields.update({f"{name}_kernel_mean_us": round(mean, 3),
                       f"{name}_kernel_min_us": round(min(durs), 3),
                       f"{name}_kernel_max_us": round(max(durs), 3),
                       f"{name}_event_mean_us": ev[name],
                       f"{name}_kv_bytes": alg[name],
                       f"{name}_kernel_frac": round(gbs / HBM_PEAK_GBS, 4)})
        if mean > ev[name]:
            out.append(f"\nWARNING: the {name} kernels' mean exceeds the events that bracket them.")
    r = rec["roofline"]
    out += ["",
            "Each call's HIP events bracket its kernel (the launch, the dispatch and the",
            "completion signal included), so the kernel mean sits at or below the event mean.",
            "",
            "The bench line of the same invocation (run under the profiler, so a little",
            "slower than an unprofiled run):",
            "",
            "    " + json.dumps({k: rec[k] for k in ("metric", "value", "unit", "steps", "warmup",
                                                   "ms_per_step")}),
            "    roofline: " + json.dumps({k: r.get(k) for k in ("achieved", "frac",
                                                                  "algorithmic_bytes_per_launch")}),
            "",
            "Fields read by bench.py (`roofline.kernel_time`), valid while the kernel sources",
            "hash to kernel_source_sha256:",
            ""]
    out += [f"{k}: {v}" for k, v in fields.items()]
    return "\n".join(out) + "\n"


def summarize_counters(fetch_csv, write_csv, bench_json, cmd):
    rec = _bench_line(bench_json)
    W, K, S0 = rec["warmup"], rec["steps"], settle_count(rec)
    det = rec["detail"]
    alg = {"verify": det["verify_kv_bytes"], "draft": det["draft_kv_bytes"]}
    res = {}
    calib = {}
    for ctr, path in (("FETCH_SIZE", fetch_csv), ("WRITE_SIZE", write_csv)):
        ds = _dispatches(_rows(path))
        copies = [d for d in ds if "bench_copy_kernel" in d["name"]]
        if not copies:
            raise SystemExit(f"{path}: no md_bench_copy dispatch to calibrate {ctr}")
        calib[ctr] = copies[-1][ctr]
        ver, dra = timed_calls(ds, W, K, S0)
        for name, calls in (("verify", ver), ("draft", dra)):
            vals = [sum(d[ctr] for d in c) for c in calls]
            res[(name, ctr)] = (sum(vals) / len(vals), sorted({_short(d["name"]) for c in calls for d in c}))
    gib = float(1 << 30)
    scale = {c: gib / (calib[c] * 1024.0) for c in calib}
    out = ["# HBM traffic of the bench's verify and draft calls (rocprofv3 counters)",
           "",
           f"Workload: {WORKLOAD} -- Llama-3.1-8B layer shape, B = 64, S = 32768, 16-token pages,",
           "gamma = 4, draft 16 sinks + 1008 window, bf16.  One MI355X (gfx950).",
           "",
           "Commands (from /tmp with TMPDIR=/tmp; R = the repository root), one pass per counter:",
           ""]
    out += [f"    {c}" for c in cmd.split(" ;; ")]
    out += ["",
            "Calibration: bench.py copies exactly 1 GiB with md_bench_copy (1,073,741,824 B read",
            f"and written).  FETCH_SIZE read {calib['FETCH_SIZE']:.0f} KiB for it and WRITE_SIZE "
            f"{calib['WRITE_SIZE']:.0f} KiB, so",
            f"bytes = KiB x 1024 x scale with scale_fetch = {scale['FETCH_SIZE']:.5f}, "
            f"scale_write = {scale['WRITE_SIZE']:.5f}.",
            "",
            "The timed calls are picked as in the kernel-trace summary (the settling verify calls,",
            "the warm-up steps, then the timed steps of a verify and a draft call each; here",
            f"{S0} settling calls, W = {W}, K = {K}); each row averages over the K timed calls.",
            "",
            "| call | kernel | FETCH_SIZE KiB | WRITE_SIZE KiB | HBM bytes read | HBM bytes written | algorithmic K/V bytes | read / algorithmic |",
            "|---|---|---|---|---|---|---|---|"]
    fields = {"kernel_source_sha256": kernel_source_sha256(), "settle": S0, "warmup": W, "steps": K,
              "scale_fetch": round(scale["FETCH_SIZE"], 6), "scale_write": round(scale["WRITE_SIZE"], 6)}
    for name in ("verify", "draft"):
        f_kib, kn = res[(name, "FETCH_SIZE")]
        w_kib, _ = res[(name, "WRITE_SIZE")]
        fb, wb = f_kib * 1024 * scale["FETCH_SIZE"], w_kib * 1024 * scale["WRITE_SIZE"]
        out.append(f"| {name} | {' + '.join('`%s`' % k for k in kn)} | {f_kib:.0f} | {w_kib:.0f} | "
                   f"{fb:.4e} | {wb:.4e} | {alg[name]:.4e} | {fb / alg[name]:.4f} |")
        fields[f"{name}_fetch_bytes_per_launch"] = round(fb)
        fields[f"{name}_write_bytes_per_launch"] = round(wb)
        fields[f"{name}_kv_bytes"] = alg[name]
    out += ["",
            "Fields read by bench.py (`roofline.traffic` = verify fetch + write bytes per",
            "launch), valid while the kernel sources hash to kernel_source_sha256:", ""]
    out += [f"{k}: {v}" for k, v in fields.items()]
    return "\n".join(out) + "\n"


def summarize_mfma(csv_path, bench_json, cmd):
    rec = _bench_line(bench_json)
    W, K, S0 = rec["warmup"], rec["steps"], settle_count(rec)
    cfg = rec["config"]
    ds = _dispatches(_rows(csv_path))
    ver, dra = timed_calls(ds, W, K, S0)
    tr = read_trace()
    out = ["# MFMA use of the bench's verify and draft calls (rocprofv3 counters)",
           "",
           f"Workload: {WORKLOAD} (as the other profiles).  One MI355X (gfx950): 256 CUs,",
           "1024 SIMDs, dense bf16 MFMA peak 2.5 PFLOP/s.",
           "",
           "Command (from /tmp with TMPDIR=/tmp; R = the repository root):",
           "",
           f"    {cmd}",
           "",
           "MfmaFlopsBF16 = SQ_INSTS_VALU_MFMA_MOPS_BF16 x 512; MfmaUtil = sum of",
           "SQ_VALU_MFMA_BUSY_CYCLES / (GRBM_GUI_ACTIVE x SIMDs) x 100 (rocprofv3's own",
           "definitions).  The rate divides the FLOP per launch by the timed kernel mean of",
           "the kernel-trace summary.  By design each call issues, per (sequence, kv head)",
           "and visible key (rounded up to 32-token tiles), 2 contractions x 2 FLOP x d x the",
           "padded query rows (16 per 16-row tile).",
           "",
           "| call | kernel | FLOP per launch | by design | kernel mean us | bf16 TFLOP/s | frac of 2.5 PFLOP/s | MfmaUtil % |",
           "|---|---|---|---|---|---|---|---|"]
    G = cfg["Hq"] // cfg["Hkv"]
    rows_pad = -(-(G * (cfg["gamma"] + 1)) // 16) * 16
    per_key = 2 * 2 * cfg["head_dim"] * rows_pad
    u_draft = min(cfg["S"], cfg["n_sink"] + cfg["gamma"] + cfg["window"])  # sinks + union of windows
    design = {"verify": cfg["B"] * cfg["Hkv"] * (-(-cfg["S"] // 32) * 32) * per_key,
              "draft": cfg["B"] * cfg["Hkv"] * (-(-u_draft // 32) * 32) * per_key}
    fields = {"kernel_source_sha256": kernel_source_sha256(), "settle": S0, "warmup": W,
              "steps": K}
    for name, calls in (("verify", ver), ("draft", dra)):
        fl = sum(sum(d.get("MfmaFlopsBF16", 0.0) for d in c) for c in calls) / len(calls)
        ut = sum(sum(d.get("MfmaUtil", 0.0) for d in c) for c in calls) / len(calls)
        kn = sorted({_short(d["name"]) for c in calls for d in c})
        mean = tr[f"{name}_kernel_mean_us"] if tr else float("nan")
        tf = fl / (mean * 1e-6) / 1e12
        out.append(f"| {name} | {' + '.join('`%s`' % k for k in kn)} | {fl:.4e} | {design[name]:.4e} | "
                   f"{mean:.2f} | {tf:.1f} | {tf / MFMA_BF16_PEAK_TFLOPS:.4f} | {ut:.2f} |")
        fields.update({f"{name}_mfma_flop_per_launch": f"{fl:.6e}",
                       f"{name}_mfma_tflops": round(tf, 2), f"{name}_mfma_busy_pct": round(ut, 3)})
    passes = {}
    for d in ds:
        if "snapkv_pass_kernel" in d["name"]:
            passes.setdefault(_short(d["name"]), []).append(d)
    if passes:
        out += ["", "The SnapKV passes of the same run (64 prompts of 32768 tokens, 128 observation rows a",
                "kv head; 2 FLOP x d per row and key), means over every dispatch, the rate by the",
                "dispatch's own duration under the counters:", "",
                "| kernel | dispatches | FLOP per launch | us | bf16 TFLOP/s | MfmaUtil % |",
                "|---|---|---|---|---|---|"]
        for k, dl in passes.items():
            fl = sum(d.get("MfmaFlopsBF16", 0.0) for d in dl) / len(dl)
            us = sum(d["end"] - d["start"] for d in dl) / len(dl) / 1e3
            ut = sum(d.get("MfmaUtil", 0.0) for d in dl) / len(dl)
            out.append(f"| `{k}` | {len(dl)} | {fl:.4e} | {us:.1f} | {fl / us / 1e6:.1f} | {ut:.2f} |")
    out += ["", "Fields read by bench.py (`roofline.mfma`), valid while the kernel sources hash to",
            "kernel_source_sha256:", ""]
    out += [f"{k}: {v}" for k, v in fields.items()]
    return "\n".join(out) + "\n"


def input_sha256(c, piece=1 << 28):
    """SHA-256 of each seeded input tensor's bytes (the whole K and V pools
    included), so that two runs can be shown to have timed the same data.
    Tensors are copied to the host a piece at a time."""
    import torch

    out = {}
    for name in ("q", "k", "v", "kv_lens", "page_table"):
        t = c.get(name)
        if t is None:
            continue
        flat = t.detach().contiguous().view(-1).view(torch.uint8)
        h = hashlib.sha256()
        for s in range(0, flat.numel(), piece):
            h.update(flat[s:s + piece].cpu().numpy().tobytes())
        out[name] = h.hexdigest()
    return out


def cpu_baseline(c, w, budget_s=15.0, batch=32):
    """The fp64 oracle (as it stands) on a bounded sample of the same workload:
    verify + draft over (sequence, kv head) units in seeded random order,
    batch by batch until `budget_s` of oracle time or every unit is done."""
    import numpy as np

    import oracle
    from paper_2408_11049_amd import workloads as wl

    threads = oracle.default_threads()

    def run(units):
        qs, ks, vs, lens = [], [], [], []
        for b, hk in units:
            q, k, v, S = wl.gather_unit(c, b, hk)
            qs.append(q), ks.append(k), vs.append(v), lens.append(int(S[0]))
        Smax = max(lens)
        kk = np.zeros((len(units), Smax, 1, w.d), dtype=ks[0].dtype)
        vv = np.zeros_like(kk)
        for i, (k, v) in enumerate(zip(ks, vs)):
            kk[i, : k.shape[1]] = k[0]
            vv[i, : v.shape[1]] = v[0]
        qq = np.concatenate(qs, axis=0)
        ll = np.array(lens, dtype=np.int32)
        t0 = time.perf_counter()
        oracle.verify(qq, kk, vv, ll, nthreads=threads)
        oracle.draft(qq, kk, vv, ll, w.n_sink, w.window, nthreads=threads)
        dt = time.perf_counter() - t0
        # K/V bytes of one kv head: the per-call formulas divided by Hkv.
        by = (kv_bytes(w, lens, "verify", w.q_len) + kv_bytes(w, lens, "draft", w.q_len)) // w.Hkv
        return dt, by

    order = np.random.default_rng(0).permutation(w.B * w.Hkv)
    units = [(int(x) // w.Hkv, int(x) % w.Hkv) for x in order]
    total_t, total_b, done = 0.0, 0, 0
    while done < len(units) and total_t < budget_s:
        dt, by = run(units[done: done + batch])
        total_t += dt
        total_b += by
        done += min(batch, len(units) - done)
    model = None
    if os.path.exists("/proc/cpuinfo"):
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    try:
        affinity = len(os.sched_getaffinity(0))
    except AttributeError:
        affinity = None
    return {"value": total_b / total_t / 1e9, "unit": "GB/s", "cores": threads, "kind": "oracle",
            "cpu_model": model, "host_cpus": os.cpu_count(), "cpus_available": affinity,
            "thread_rule": "one per CPU this process may use, at most 16 (one GPU's share "
                           "of a shared GPU host)",
            "sample": f"{done} of {len(units)} (sequence, kv head) units of {WORKLOAD} in seeded "
                      f"random order, verify + draft, {total_t:.1f} s of fp64 oracle time"}


def cpu_oracle_extras(c, w, logits, draft_tok, q_obs, n_obs, t_accept_us, t_votes_us):
    """The oracle beside the steps around verification: greedy acceptance
    over the whole logits tensor, and SnapKV votes of a few sampled (prompt,
    kv head) units scaled to the whole batch."""
    import numpy as np

    import oracle
    import oracle.sdstep as sd
    from paper_2408_11049_amd import workloads as wl

    host_logits = wl.to_host_bits(logits)
    host_draft = draft_tok.cpu().numpy()
    t0 = time.perf_counter()
    sd.greedy_accept(host_logits, host_draft)
    t_acc = time.perf_counter() - t0
    units = [(0, 0), (w.B // 2, w.Hkv // 2), (w.B - 1, w.Hkv - 1)]
    G = w.Hq // w.Hkv
    t_votes = 0.0
    for b, hk in units:
        q = wl.to_host_bits(q_obs[b: b + 1, :, hk * G: (hk + 1) * G])
        _, k, _, S = wl.gather_unit(c, b, hk)
        t0 = time.perf_counter()
        oracle.snapkv_votes(q, k, S, pool=5)
        t_votes += time.perf_counter() - t0
    t_votes_all = t_votes / len(units) * w.B * w.Hkv
    # The oracle on one thread over the two smallest workloads: the whole of
    # tiny_f32, and two of llama8b_b32_s8k's 32 sequences (all 8 kv heads).
    one = {}
    for name, B in (("tiny_f32", None), ("llama8b_b32_s8k", 2)):
        ww = wl.WORKLOADS[name]
        cc = wl.make_case(B=B or ww.B, q_len=ww.q_len, Hq=ww.Hq, Hkv=ww.Hkv, d=ww.d,
                          kv_lens=[ww.S] * (B or ww.B), dtype=ww.dtype, seed=ww.seed_base,
                          device="cpu", nan_pad=False)
        q, k, v = (wl.to_host_bits(cc[x]) for x in ("q", "k", "v"))
        lens = cc["kv_lens_np"]
        t0 = time.perf_counter()
        oracle.verify(q, k, v, lens, nthreads=1)
        oracle.draft(q, k, v, lens, ww.n_sink, ww.window, nthreads=1)
        dt = time.perf_counter() - t0
        by = kv_bytes(ww, lens, "verify", ww.q_len) + kv_bytes(ww, lens, "draft", ww.q_len)
        one[f"oracle_one_thread_{name}"] = {
            "gbs": round(by / dt / 1e9, 4), "s": round(dt, 3),
            "sample": "whole workload" if B is None else f"{B} of {ww.B} sequences"}
    return {**one,
            "greedy_accept_s (numpy, one thread, whole logits)": round(t_acc, 3),
            "greedy_accept_gpu_speedup": round(t_acc / (t_accept_us * 1e-6), 1),
            "snapkv_votes_s (fp64 C, one thread, 3 sampled units scaled to all)": round(t_votes_all, 2),
            "snapkv_votes_gpu_speedup": round(t_votes_all / (t_votes_us * 1e-6), 1)}


def settle(fn, flush_fn, ms, sync, min_calls=5):
    """Untimed: eviction + fn back to back for at least `ms` milliseconds of
    wall time and at least `min_calls` calls (ms = 0: exactly min_calls, so a
    profiled run's dispatch ordinals do not depend on its speed),
    synchronising every few calls.  After
    host-side setup or a phase of short calls leaves HBM lightly loaded, the
    first ~15-20 ms of HBM-bound launches run up to ~20% slower on MI355X
    (measured: a ragged B = 64 verify falls from 1161 us to ~950 us over its
    first 15 calls, then stays); timed regions start from the steady state of
    a serving loop instead.  Returns the number of calls."""
    n = 0
    t_end = time.perf_counter() + ms * 1e-3
    while n < min_calls or (ms > 0 and time.perf_counter() < t_end):
        flush_fn()
        fn()
        n += 1
        if n % 4 == 0:
            sync()
    sync()
    return n


def config_table(w_names, dev, timed, verbose=True, settle_fn=None):
    """Cold-cache medians (p10, p50, p90 of 10 calls) of every configuration in
    the workload list: verify and draft at q_len = gamma + 1 and 1, t_step,
    t_SD = gamma t_draft(1) + t_verify (the attention part of Eq. 2's step
    time), the ratio t_verify(gamma + 1) / t_verify(1) (Sec. 3.2 predicts ~1
    where the KV cache dominates), K/V GB/s and fractions of 8 TB/s."""
    import torch

    import paper_2408_11049_amd as md
    from paper_2408_11049_amd import workloads as wl

    table = {}
    for name in w_names:
        w = wl.WORKLOADS[name]
        log(f"[bench] config {name}")
        c = wl.make_workload(w, device=dev)
        lens, L = c["kv_lens_np"], w.q_len
        q1 = c["q"][:, :1].contiguous()
        common = dict(max_kv_len=c["max_kv_len"], page_table=c["page_table"])
        need = max(md.md_workspace_bytes(q, c["k"], c["v"], c["kv_lens"], mode=m, n_sink=w.n_sink,
                                         window=w.window, **common)
                   for q in (c["q"], q1) for m in (0, 1))
        ws = torch.empty(max(need, 256), dtype=torch.uint8, device=dev) if need else None
        o, o1 = torch.empty_like(c["q"]), torch.empty_like(q1)
        kw = dict(return_lse=False, workspace=ws, **common)
        calls = {
            "verify": lambda: md.md_verify_attn(c["q"], c["k"], c["v"], c["kv_lens"], out=o, **kw),
            "verify_qlen1": lambda: md.md_verify_attn(q1, c["k"], c["v"], c["kv_lens"], out=o1, **kw),
            "draft": lambda: md.md_draft_attn(c["q"], c["k"], c["v"], c["kv_lens"], w.n_sink,
                                              w.window, out=o, **kw),
            "draft_qlen1": lambda: md.md_draft_attn(q1, c["k"], c["v"], c["kv_lens"], w.n_sink,
                                                    w.window, out=o1, **kw),
        }
        for fn in calls.values():
            fn()
        n_settle = settle_fn(calls["verify"]) if settle_fn else 0
        t = {k: timed(fn, n=10, stats=True) for k, fn in calls.items()}
        by = {"verify": kv_bytes(w, lens, "verify", L), "verify_qlen1": kv_bytes(w, lens, "verify", 1),
              "draft": kv_bytes(w, lens, "draft", L), "draft_qlen1": kv_bytes(w, lens, "draft", 1)}
        row = {"shape": f"B={w.B} Hq={w.Hq} Hkv={w.Hkv} d={w.d} gamma={w.gamma} "
                        f"S={w.S or f'{w.S_lo}..{w.S_hi}'} sinks+window={w.n_sink}+{w.window} "
                        f"{w.dtype} {'paged ' + str(w.page_size) if w.page_size else 'contiguous'}"}
        for k in calls:
            p50 = t[k][1]
            row[f"t_{k}_us_p10_p50_p90"] = t[k]
            row[f"{k}_kv_bytes"] = by[k]
            row[f"{k}_gbs"] = round(by[k] / (p50 * 1e-6) / 1e9, 1)
            row[f"{k}_frac"] = round(by[k] / (p50 * 1e-6) / 1e9 / HBM_PEAK_GBS, 4)
        row["t_step_us (verify + draft)"] = round(t["verify"][1] + t["draft"][1], 2)
        row["t_sd_us (gamma x draft_qlen1 + verify)"] = round(w.gamma * t["draft_qlen1"][1] + t["verify"][1], 2)
        row["verify_ratio_qlen_gamma1_vs_1"] = round(t["verify"][1] / t["verify_qlen1"][1], 4)
        row["settle_calls (untimed verify calls first, >= 60 ms)"] = n_settle
        table[name] = row
        if verbose:
            log(f"[bench]   verify {t['verify'][1]:.1f} us ({row['verify_frac']:.3f})  draft "
                f"{t['draft'][1]:.1f} us ({row['draft_frac']:.3f})  draft(1) {t['draft_qlen1'][1]:.1f} us")
        del c, ws, o, o1, q1
        torch.cuda.empty_cache()
    return table


LATENCY_CASES = [("llama8b_b32_s8k", "draft"), ("llama8b_b32_s8k", "draft_qlen1"),
                 ("llama70b_b16_s128k", "draft"), ("llama70b_b16_s128k", "draft_qlen1"),
                 ("llama8b_b64_s32k_paged", "draft")]


def latency_breakdown(dev, warm=3, reps=10):
    """Where a short call's time goes: per case, `warm` untimed calls, then
    `reps` calls timed by HIP events, then `reps` calls through
    md_bench_attn_stamps (the same launch, each workgroup stamping the GPU's
    100 MHz wall clock at its start, after its first tile, at the end of its
    main loop and at its end).  Every call follows a cache eviction.  Run
    under rocprofv3 --kernel-trace, the trace adds each timed call's kernel
    duration (bench.py --summarize latency)."""
    import numpy as np
    import torch

    import paper_2408_11049_amd as md
    from paper_2408_11049_amd import workloads as wl

    lib = md.load_library()
    stream = torch.cuda.current_stream(dev)
    sh = md.ctypes.c_void_p(stream.cuda_stream)
    buf = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    sink = torch.zeros(4, dtype=torch.float32, device=dev)

    def evict():
        md._check(lib.md_bench_evict(md.ctypes.c_void_p(buf.data_ptr()), buf.numel(),
                                     md.ctypes.c_void_p(sink.data_ptr()), sh))

    out, cache = [], {}
    for name, call in LATENCY_CASES:
        w = wl.WORKLOADS[name]
        if name not in cache:
            cache.clear()
            torch.cuda.empty_cache()
            cache[name] = wl.make_workload(w, device=dev)
        c = cache[name]
        q = c["q"][:, :1].contiguous() if call.endswith("qlen1") else c["q"]
        common = dict(max_kv_len=c["max_kv_len"], page_table=c["page_table"])
        need = md.md_workspace_bytes(q, c["k"], c["v"], c["kv_lens"], mode=1, n_sink=w.n_sink,
                                     window=w.window, **common)
        ws = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
        o = torch.empty_like(q)

        def run():
            md.md_draft_attn(q, c["k"], c["v"], c["kv_lens"], w.n_sink, w.window, out=o,
                             return_lse=False, workspace=ws, **common)

        for _ in range(warm):
            evict()
            run()
        ev = []
        for _ in range(reps):
            evict()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream); run(); b.record(stream)
            torch.cuda.synchronize()
            ev.append(a.elapsed_time(b) * 1e3)
        phases = {k: [] for k in ("start_spread", "first_tile", "loop", "epilogue", "span")}
        for _ in range(reps):
            evict()
            _, st = md.md_bench_attn_stamps(1, q, c["k"], c["v"], c["kv_lens"], w.n_sink, w.window,
                                            out=o, workspace=ws, **common)
            torch.cuda.synchronize()
            x = st.cpu().numpy().astype(np.int64)
            x = x[x[:, 3] > 0]
            t0 = x[:, 0].min()
            phases["start_spread"].append((x[:, 0].max() - t0) / 100.0)
            phases["first_tile"].append(float(np.median(x[:, 1] - x[:, 0])) / 100.0)
            phases["loop"].append(float(np.median(x[:, 2] - x[:, 1])) / 100.0)
            phases["epilogue"].append(float(np.median(x[:, 3] - x[:, 2])) / 100.0)
            phases["span"].append((x[:, 3].max() - t0) / 100.0)
        q_len = q.shape[1]
        out.append({"workload": name, "call": call, "q_len": q_len, "warm": warm, "reps": reps,
                    "kv_bytes": kv_bytes(w, c["kv_lens_np"], "draft", q_len),
                    "workgroups": int(len(x)), "split": bool(need),
                    "event_us": [round(v, 2) for v in ev],
                    "stamps_us_median": {k: round(float(np.median(v)), 2) for k, v in phases.items()}})
        log(f"[bench] {name} {call}: event {np.median(ev):.1f} us, stamps "
            f"{out[-1]['stamps_us_median']}")
    return out


def summarize_latency(csv_path, bench_json, cmd):
    rec = None
    for line in open(bench_json):
        if line.strip().startswith("{") and '"latency"' in line:
            rec = json.loads(line)
    if rec is None:
        raise SystemExit(f"no latency line in {bench_json}")
    calls = attention_calls(_dispatches(_rows(csv_path)))
    out = ["# Where a draft call's time goes (rocprofv3 kernel trace + workgroup stamps)",
           "",
           "Draft calls (sinks + window, at q_len = gamma + 1 and 1) of the llama8b_b32_s8k",
           "(B = 32, S = 8192, 16 + 496), llama70b_b16_s128k (B = 16, S = 131072, 64 + 1984) and",
           "bench (B = 64, S = 32768 paged, 16 + 1008) workloads, each after a 1 GiB cache",
           "eviction.  One MI355X (gfx950).",
           "",
           "Command (from /tmp with TMPDIR=/tmp; R = the repository root):",
           "",
           f"    {cmd}",
           "",
           "and this summary from its trace and stdout by",
           "",
           "    python3 $R/bench.py --summarize latency --csv $R/gpurun_out/prof/lat/bench_kernel_trace.csv "
           "--bench-json $R/gpurun_out/prof/lat_bench.json --cmd \"<the command above>\"",
           "",
           "Per case the run makes `warm` untimed calls, `reps` event-timed calls and `reps`",
           "stamped calls (md_bench_attn_stamps: the same launch, each workgroup recording the",
           "100 MHz wall clock at its start, after its first K/V tile, at the end of its main",
           "loop and at its end).  The kernel column is the trace's duration of the event-timed",
           "calls (attention kernel, plus the merge kernel of a split plan); launch overhead is",
           "event minus kernel.  Stamp columns are medians over workgroups and calls.",
           "",
           "| workload | call | K/V bytes | workgroups | event us | kernel us | of which merge us | launch overhead us | first tile us | main loop us | epilogue us | span (stamps) us | K/V GB/s (event) | frac (event) | frac (kernel) |",
           "|---|---|---|---|---|---|---|---|---|---|---|---|---|---|---|"]
    i = 0
    for case in rec["latency"]:
        n = case["warm"] + 2 * case["reps"]
        mine = calls[i: i + n]
        i += n
        timed = mine[case["warm"]: case["warm"] + case["reps"]]
        kern = sorted(sum(d["end"] - d["start"] for d in c) / 1e3 for c in timed)
        merge = sorted(sum(d["end"] - d["start"] for d in c[1:]) / 1e3 for c in timed)
        km, mm = kern[len(kern) // 2], merge[len(merge) // 2]
        ev = sorted(case["event_us"])[len(case["event_us"]) // 2]
        st = case["stamps_us_median"]
        by = case["kv_bytes"]
        out.append(f"| {case['workload']} | {case['call']} | {by} | {case['workgroups']} | {ev:.2f} | "
                   f"{km:.2f} | {mm:.2f} | {ev - km:.2f} | {st['first_tile']:.2f} | {st['loop']:.2f} | "
                   f"{st['epilogue']:.2f} | {st['span']:.2f} | {by / (ev * 1e-6) / 1e9:.0f} | "
                   f"{by / (ev * 1e-6) / 1e9 / HBM_PEAK_GBS:.3f} | {by / (km * 1e-6) / 1e9 / HBM_PEAK_GBS:.3f} |")
    out += ["", f"kernel_source_sha256: {kernel_source_sha256()}"]
    return "\n".join(out) + "\n"


PAGED_AB_CASES = ["paged (seeded random page order)", "paged (pages in sequence order)",
                  "contiguous"]


def paged_ab(dev, warm=2, reps=10):
    """The bench-shape verify over the same K/V three ways, interleaved in one
    process: through the workload's page table (pages in seeded random order),
    through a table whose pages lie in sequence order, and from a contiguous
    [B, S, Hkv, d] copy.  Each call follows a cache eviction; `warm` rounds
    are untimed.  Run under rocprofv3 --pmc, the counter summary attributes
    translation misses and read latency to each case."""
    import numpy as np
    import torch

    import paper_2408_11049_amd as md
    from paper_2408_11049_amd import workloads as wl

    lib = md.load_library()
    stream = torch.cuda.current_stream(dev)
    sh = md.ctypes.c_void_p(stream.cuda_stream)
    buf = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    sink = torch.zeros(4, dtype=torch.float32, device=dev)
    w = wl.WORKLOADS[WORKLOAD]
    c = wl.make_workload(w, device=dev)
    B, S, ps = w.B, w.S, w.page_size
    pt = c["page_table"].long().view(-1)
    kc = c["k"][pt].view(B, S, w.Hkv, w.d)
    vc = c["v"][pt].view(B, S, w.Hkv, w.d)
    seq_table = torch.arange(B * (S // ps), device=dev, dtype=torch.int32).view(B, -1)
    kp, vp = kc.view(-1, ps, w.Hkv, w.d), vc.view(-1, ps, w.Hkv, w.d)
    outs = [torch.empty_like(c["q"]) for _ in PAGED_AB_CASES]
    kw = dict(max_kv_len=S, return_lse=False)
    calls = [
        lambda: md.md_verify_attn(c["q"], c["k"], c["v"], c["kv_lens"], out=outs[0],
                                  page_table=c["page_table"], **kw),
        lambda: md.md_verify_attn(c["q"], kp, vp, c["kv_lens"], out=outs[1], page_table=seq_table,
                                  **kw),
        lambda: md.md_verify_attn(c["q"], kc, vc, c["kv_lens"], out=outs[2], **kw),
    ]
    ev = [[] for _ in calls]
    for r in range(warm + reps):
        for i, fn in enumerate(calls):
            md._check(lib.md_bench_evict(md.ctypes.c_void_p(buf.data_ptr()), buf.numel(),
                                         md.ctypes.c_void_p(sink.data_ptr()), sh))
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream); fn(); b.record(stream)
            torch.cuda.synchronize()
            if r >= warm:
                ev[i].append(a.elapsed_time(b) * 1e3)
    same = all(torch.equal(outs[0], o) for o in outs[1:])
    res = {"cases": PAGED_AB_CASES, "warm": warm, "reps": reps, "bytes": kv_bytes(w, c["kv_lens_np"], "verify", w.q_len),
           "event_us": [[round(x, 2) for x in e] for e in ev], "outputs_identical": bool(same)}
    log("[bench] paged A/B: " + ", ".join(f"{n}: {np.median(e):.1f} us" for n, e in zip(PAGED_AB_CASES, ev)))
    return res


def summarize_paged(csv_path, bench_json, cmd):
    rec = None
    for line in open(bench_json):
        if line.strip().startswith("{") and '"paged_ab"' in line:
            rec = json.loads(line)["paged_ab"]
    if rec is None:
        raise SystemExit(f"no paged_ab line in {bench_json}")
    n = len(rec["cases"])
    calls = [d for d in _dispatches(_rows(csv_path)) if "attn_partial_kernel" in d["name"]]
    per = [calls[i::n][rec["warm"]:] for i in range(n)]
    out = ["# Paged against contiguous K/V: the bench-shape verify (rocprofv3 counters)",
           "",
           f"Workload: {WORKLOAD} (B = 64, S = 32768, Hkv = 8, d = 128, bf16, gamma = 4) verified",
           "three ways over the same K/V values in one process, calls interleaved, each after a",
           "1 GiB cache eviction: through the workload's 16-token page table (seeded random page",
           "placement), through a table whose pages lie in sequence order, and from a",
           "contiguous [B, S, Hkv, d] copy.  Outputs identical in all three: "
           f"{rec['outputs_identical']}.  One MI355X (gfx950).",
           "",
           "Commands (from /tmp with TMPDIR=/tmp; R = the repository root): the times come from",
           "an unprofiled run, the counters from a second run of the same command under",
           "rocprofv3 (counter collection serialises the dispatches):",
           ""]
    out += [f"    {c}" for c in cmd.split(" ;; ")]
    out += ["",
            "| case | event median us | K/V GB/s | UTCL1 translation misses | UTCL1 translation hits | miss rate | TCP->TCC read requests | mean read latency (cycles) |",
            "|---|---|---|---|---|---|---|---|"]
    for i, name in enumerate(rec["cases"]):
        e = sorted(rec["event_us"][i])[len(rec["event_us"][i]) // 2]
        ds = per[i]
        avg = lambda k: sum(d.get(k, 0.0) for d in ds) / max(len(ds), 1)
        miss, hit = avg("TCP_UTCL1_TRANSLATION_MISS_sum"), avg("TCP_UTCL1_TRANSLATION_HIT_sum")
        req, lat = avg("TCP_TCC_READ_REQ_sum"), avg("TCP_TCC_READ_REQ_LATENCY_sum")
        out.append(f"| {name} | {e:.2f} | {rec['bytes'] / (e * 1e-6) / 1e9:.0f} | {miss:.4g} | {hit:.4g} | "
                   f"{miss / max(miss + hit, 1):.4f} | {req:.4g} | {lat / max(req, 1):.1f} |")
    out += ["", f"kernel_source_sha256: {kernel_source_sha256()}"]
    return "\n".join(out) + "\n"


CONFIG_KINDS = ["verify", "verify_qlen1", "draft", "draft_qlen1"]


def config_calls(calls, rec):
    """The timed calls of the per-configuration table, picked by ordinal: the
    table is the run's last attention work, and per configuration (in CONFIGS
    order) it makes one warm call of each kind, its settling verify calls,
    then 10 timed calls of each kind in CONFIG_KINDS order.  Returns
    {config: {kind: [call, ...]}}."""
    cfgs = rec["detail"]["configs"]
    names = [n for n in CONFIGS if n in cfgs]
    out, idx = {}, len(calls)
    for name in reversed(names):
        settle = next((int(v) for k, v in cfgs[name].items() if k.startswith("settle_calls")), 0)
        timed = calls[idx - 40: idx]
        idx -= 40 + settle + len(CONFIG_KINDS)
        if idx < 0 or len(timed) != 40:
            raise SystemExit(f"{name}: the trace holds too few attention calls for the table")
        out[name] = {k: timed[10 * i: 10 * i + 10] for i, k in enumerate(CONFIG_KINDS)}
        for k, cl in out[name].items():
            kn = {_short(c[0]["name"]) for c in cl}
            if len(kn) != 1:
                raise SystemExit(f"{name} {k}: the picked calls run different kernels: {sorted(kn)}")
    return out


def summarize_configs(csv_path, bench_json, cmd):
    """Kernel-trace times of the per-configuration table's timed calls next to
    the event-timed medians of the same bench line."""
    import numpy as np

    rec = _bench_line(bench_json)
    cfgs = rec["detail"]["configs"]
    per = config_calls(attention_calls(_dispatches(_rows(csv_path))), rec)
    out = ["# Kernel timing of the per-configuration table (rocprofv3 kernel trace)",
           "",
           "Every configuration of the workload list, verify and draft at q_len = gamma + 1",
           "and 1, each call after a 1 GiB cache eviction, 10 timed calls per kind after the",
           "configuration's settling calls.  One MI355X (gfx950).",
           "",
           "Command (from /tmp with TMPDIR=/tmp; R = the repository root); its stdout is the",
           "bench line whose detail.configs gives the event medians:",
           "",
           f"    {cmd}",
           "",
           "Selection: the table is the run's last attention work; per configuration it makes",
           "one warm call of each kind, its settling verify calls (their count is in the bench",
           "line), then 10 timed calls of verify, one-token verify, draft and one-token draft,",
           "so the summary walks back from the last attention dispatch.  A merge dispatch that",
           "follows a call (split plans) counts with it.  Under the tracer the event medians",
           "run a little slower than unprofiled.",
           "",
           "| configuration | call | kernel | kernel median us | event median us | kernel / event | K/V bytes | frac of 8 TB/s (kernel) | frac (event) |",
           "|---|---|---|---|---|---|---|---|---|"]
    for name in CONFIGS:
        if name not in per:
            continue
        row = cfgs[name]
        for k in CONFIG_KINDS:
            durs = [sum(d["end"] - d["start"] for d in c) / 1e3 for c in per[name][k]]
            km = float(np.median(durs))
            ev = float(row[f"t_{k}_us_p10_p50_p90"][1])
            by = float(row[f"{k}_kv_bytes"])
            kn = " + merge" if any(len(c) > 1 for c in per[name][k]) else ""
            out.append(f"| {name} | {k} | `{_short(per[name][k][0][0]['name'])}`{kn} | {km:.2f} | {ev:.2f} | "
                       f"{km / ev:.3f} | {by:.4g} | {by / (km * 1e-6) / 1e9 / HBM_PEAK_GBS:.4f} | "
                       f"{by / (ev * 1e-6) / 1e9 / HBM_PEAK_GBS:.4f} |")
    out += ["", f"kernel_source_sha256: {kernel_source_sha256()}"]
    return "\n".join(out) + "\n"


def summarize_config_counters(fetch_csv, write_csv, fetch_json, write_json, cmd):
    """HBM traffic of the per-configuration table's timed calls: FETCH_SIZE and
    WRITE_SIZE per call (attention plus merge), scaled by a copy of known
    size in the same run, against the algorithmic K/V bytes."""
    res, calib, kernels = {}, {}, {}
    for ctr, path, bj in (("FETCH_SIZE", fetch_csv, fetch_json), ("WRITE_SIZE", write_csv, write_json)):
        rec = _bench_line(bj)
        ds = _dispatches(_rows(path))
        copies = [d for d in ds if "bench_copy_kernel" in d["name"]]
        if not copies:
            raise SystemExit(f"{path}: no md_bench_copy dispatch to calibrate {ctr}")
        calib[ctr] = copies[-1][ctr]
        for name, kinds in config_calls(attention_calls(ds), rec).items():
            for k, cl in kinds.items():
                res[(name, k, ctr)] = sum(sum(d[ctr] for d in c) for c in cl) / len(cl)
                kernels[(name, k)] = _short(cl[0][0]["name"]) + (" + merge" if any(len(c) > 1 for c in cl) else "")
        cfgs = rec["detail"]["configs"]
    gib = float(1 << 30)
    scale = {c: gib / (calib[c] * 1024.0) for c in calib}
    out = ["# HBM traffic of the per-configuration table (rocprofv3 counters)",
           "",
           "Every configuration of the workload list, verify and draft at q_len = gamma + 1",
           "and 1, each call after a 1 GiB cache eviction.  One MI355X (gfx950).  The timed",
           "calls are picked as in the per-configuration kernel trace (by ordinal, walking back",
           "from the last attention dispatch, with each run's own settling counts).",
           "",
           "Commands (from /tmp with TMPDIR=/tmp; R = the repository root):",
           "",
           f"    {cmd}",
           "",
           f"Calibration: a 1 GiB copy in each run read FETCH_SIZE = {calib['FETCH_SIZE']:.0f} KiB and",
           f"WRITE_SIZE = {calib['WRITE_SIZE']:.0f} KiB, so bytes = KiB x 1024 x scale with",
           f"scale_fetch = {scale['FETCH_SIZE']:.5f}, scale_write = {scale['WRITE_SIZE']:.5f}.",
           "",
           "| configuration | call | kernel | HBM bytes read | HBM bytes written | algorithmic K/V bytes | read / algorithmic |",
           "|---|---|---|---|---|---|---|"]
    for name in CONFIGS:
        if (name, "verify") not in kernels:
            continue
        for k in CONFIG_KINDS:
            rd = res[(name, k, "FETCH_SIZE")] * 1024 * scale["FETCH_SIZE"]
            wr = res[(name, k, "WRITE_SIZE")] * 1024 * scale["WRITE_SIZE"]
            alg = float(cfgs[name][f"{k}_kv_bytes"])
            out.append(f"| {name} | {k} | `{kernels[(name, k)]}` | {rd:.4g} | {wr:.4g} | {alg:.4g} | "
                       f"{rd / alg:.4f} |")
    out += ["", f"kernel_source_sha256: {kernel_source_sha256()}"]
    return "\n".join(out) + "\n"


LDS_COUNTERS = ["SQ_LDS_BANK_CONFLICT", "SQ_LDS_IDX_ACTIVE", "SQ_LDS_ADDR_CONFLICT",
                "SQ_LDS_UNALIGNED_STALL", "SQ_INSTS_LDS", "SQ_WAIT_INST_LDS", "SQ_ACTIVE_INST_LDS"]


# The prefill-time kernels of the bench line: the SnapKV passes and selection
# and the gather of the selected rows into a draft cache of their own.
PREFILL_KERNELS = [
    ("snapkv_pass_kernel", (", 0, 64", ", 0>("), "softmax statistics over K", "k_once"),
    ("snapkv_lse_kernel", ("",), "merge chunk statistics", None),
    ("snapkv_pass_kernel", (", 1, 64", ", 1>("), "votes (K again, votes written)", "k_once"),
    ("snapkv_select", ("",), "pool, radix select, compaction", "votes"),
    ("kv_gather", ("",), "listed rows into a draft cache", "gather"),
]


def summarize_prefill(trace_csv, fetch_csv, write_csv, bench_json, cmd):
    """Kernel times (trace) and HBM bytes per dispatch (FETCH_SIZE / WRITE_SIZE
    scaled by the run's 1 GiB copy) of the SnapKV and gather kernels."""
    rec = _bench_line(bench_json)
    det = rec["detail"]
    k_once = det["snapkv_votes_k_bytes (two passes over K)"] / 2
    alg = {"k_once": (k_once, "K once"), "gather": (det["kv_gather_bytes (read + write)"] / 2,
                                                    "the listed K/V rows once"),
           "votes": (None, "the votes once")}
    trace = _dispatches(_rows(trace_csv))
    ctr = {}
    calib = {}
    for c, path in (("FETCH_SIZE", fetch_csv), ("WRITE_SIZE", write_csv)):
        ds = _dispatches(_rows(path))
        calib[c] = [d for d in ds if "bench_copy_kernel" in d["name"]][-1][c]
        ctr[c] = ds
    gib = float(1 << 30)
    scale = {c: gib / (calib[c] * 1024.0) for c in calib}

    def pick(ds, key, subs):
        return [d for d in ds if key in d["name"] and any(s in d["name"] for s in subs)]

    votes_written = None
    rows = []
    for key, sub, role, a in PREFILL_KERNELS:
        tr = pick(trace, key, sub)
        if not tr:
            continue
        us = [(d["end"] - d["start"]) / 1000.0 for d in tr]
        rd = [d["FETCH_SIZE"] * 1024 * scale["FETCH_SIZE"] for d in pick(ctr["FETCH_SIZE"], key, sub)]
        wr = [d["WRITE_SIZE"] * 1024 * scale["WRITE_SIZE"] for d in pick(ctr["WRITE_SIZE"], key, sub)]
        r_b, w_b = sum(rd) / len(rd), sum(wr) / len(wr)
        if key == "snapkv_pass_kernel" and ", 1>(" in sub:
            votes_written = w_b
        rows.append((sorted({_short(d["name"]) for d in tr}), role, len(us), sum(us) / len(us),
                     min(us), max(us), r_b, w_b, a))
    out = ["# SnapKV selection and the gathered draft cache at prefill (rocprofv3)",
           "",
           f"Workload: the prompts of {WORKLOAD} -- Llama-3.1-8B heads (Hq = 32, Hkv = 8,",
           "d = 128), B = 64 prompts of 32768 tokens in 16-token pages, bf16 K/V; 32 observation",
           "queries (the prompt's last positions), pooling 5, budget 2049 (2017 selected + 32",
           "window); the 2049 selected rows of every (prompt, kv head) gathered into a draft",
           "cache of their own.  Cold cache.  One MI355X (gfx950).",
           "",
           "Commands (from /tmp with TMPDIR=/tmp; R = the repository root): the kernel trace and",
           "the FETCH_SIZE and WRITE_SIZE passes of the attention profiles,",
           ""]
    out += [f"    {c}" for c in cmd.split(" ;; ")]
    out += ["",
            f"HBM bytes = KiB x 1024 x scale, calibrated on the run's 1 GiB copy (scale_fetch =",
            f"{scale['FETCH_SIZE']:.5f}, scale_write = {scale['WRITE_SIZE']:.5f}); means over every "
            "dispatch of the run.",
            "",
            "| kernel | role | calls | avg us | min | max | HBM read bytes | HBM write bytes | "
            "algorithmic read bytes | read / algorithmic |",
            "|---|---|---|---|---|---|---|---|---|---|"]
    for names, role, n, avg, lo, hi, r_b, w_b, a in rows:
        if a is None:
            algs, ratio = "--", "--"
        else:
            ab, what = alg[a]
            if ab is None:
                ab = votes_written
            algs, ratio = f"{ab:.4e} ({what})", f"{r_b / ab:.4f}"
        out.append(f"| {' + '.join('`%s`' % k for k in names)} | {role} | {n} | {avg:.1f} | "
                   f"{lo:.1f} | {hi:.1f} | {r_b:.4e} | {w_b:.4e} | {algs} | {ratio} |")
    out += ["",
            "bench.py's HIP events around the whole calls of the same run: votes (both passes "
            f"and the merge) {det['t_snapkv_votes_us (prefill, 32 observation queries)']:.1f} us, "
            f"selection {det['t_snapkv_select_us (pool 5, budget 2049)']:.1f} us, gather "
            f"{det['t_kv_gather_us (the 2049 listed rows into a draft cache, once per prompt)']:.1f} us "
            "(under the profiler).",
            "",
            "Reading: both SnapKV passes read K exactly once each but run below the HBM rate:",
            "a wave of the bf16 passes owns 32 rows x 32 keys of a tile that the workgroup's",
            "waves share through LDS, and per score pays its share of an MFMA and a multiply-add,",
            "an exponential and an add.  The selection reads the votes once; its time goes to the",
            "radix passes over keys held in registers.  The gather reads scattered 256 B rows and",
            "stores them around the caches, so that nothing is left for the next launch to write",
            "back.  All of it runs once per prompt, at prefill."]
    return "\n".join(out) + "\n"


# The kernels around verification in the bench line, told apart by grid size
# (work-items): the (gamma+1)-token append into the paged cache, the one-token
# appends of the engine-shaped steps, both acceptance passes and the commit.
def _grid(d):
    return int(d.get("grid", 0))


def summarize_steps(trace_csv, fetch_csv, write_csv, bench_json, cmd):
    """Kernel times (trace) and HBM bytes per dispatch of the step kernels,
    grouped by (kernel, grid size); counters scaled by the run's 1 GiB copy."""
    rec = _bench_line(bench_json)
    det = rec["detail"]

    def load(path):
        out = []
        for r in _rows(path):
            g = r.get("Grid_Size_X") or r.get("Grid_Size") or 0
            out.append(dict(r, _grid=int(g)))
        return out

    def dispatches(rows):
        ds = {}
        for r in rows:
            d = ds.setdefault(int(r["Dispatch_Id"]), {"name": r["Kernel_Name"], "grid": r["_grid"]})
            if r.get("Start_Timestamp"):
                d["start"], d["end"] = int(r["Start_Timestamp"]), int(r["End_Timestamp"])
            if "Counter_Name" in r:
                d[r["Counter_Name"]] = d.get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
        return [ds[k] for k in sorted(ds)]

    trace = dispatches(load(trace_csv))
    ctr, calib = {}, {}
    for c, path in (("FETCH_SIZE", fetch_csv), ("WRITE_SIZE", write_csv)):
        ds = dispatches(load(path))
        calib[c] = [d for d in ds if "bench_copy_kernel" in d["name"]][-1][c]
        ctr[c] = ds
    gib = float(1 << 30)
    scale = {c: gib / (calib[c] * 1024.0) for c in calib}
    keys = ("kv_append_kernel", "argmax_partial_kernel", "accept_kernel", "kv_commit_kernel")
    groups = {}
    for d in trace:
        if any(k in d["name"] for k in keys):
            groups.setdefault((_short(d["name"]), _grid(d)), []).append((d["end"] - d["start"]) / 1000.0)
    alg = {"argmax_partial_kernel": (det["greedy_accept_logits_bytes"], "the logits once"),
           "kv_append_kernel": (det["kv_append_bytes (read + write)"] / 2, "the new K/V rows once")}
    big_append = max((g for (n, g) in groups if "kv_append" in n), default=0)
    am = [us for (n, g), us in groups.items() if "argmax_partial_kernel" in n]
    argmax_gbs = (det["greedy_accept_logits_bytes"] / (sum(am[0]) / len(am[0])) / 1e3
                  if am else float("nan"))
    out = ["# Kernels around verification: KV append, greedy acceptance, commit (rocprofv3)",
           "",
           f"Workload: the verify step of {WORKLOAD} -- B = 64, gamma = 4 (5 tokens per",
           "sequence), Hkv = 8, d = 128, bf16 K/V in 16-token pages; fp32 verifier logits over",
           "the Llama-3 vocabulary (128256 entries) with seeded planted targets; commit into",
           "2049-entry listed draft caches plus a 1024-slot rolling ring; the engine-shaped",
           "steps append one token per draft.  Cold cache (1 GiB evicted before every timed",
           "call).  One MI355X (gfx950).",
           "",
           "Commands (from /tmp with TMPDIR=/tmp; R = the repository root): the kernel trace and",
           "the FETCH_SIZE and WRITE_SIZE passes of the attention profiles,",
           ""]
    out += [f"    {c}" for c in cmd.split(" ;; ")]
    out += ["",
            f"HBM bytes = KiB x 1024 x scale, calibrated on the run's 1 GiB copy (scale_fetch =",
            f"{scale['FETCH_SIZE']:.5f}, scale_write = {scale['WRITE_SIZE']:.5f}); means over the "
            "dispatches of each (kernel, grid size).",
            "",
            "| kernel | work-items | calls | avg us | min | max | HBM read bytes | HBM write bytes | "
            "algorithmic read bytes | read / algorithmic |",
            "|---|---|---|---|---|---|---|---|---|---|"]
    for (name, grid), us in sorted(groups.items()):
        def mean(c):
            v = [d[c] * 1024 * scale[c] for d in ctr[c] if _short(d["name"]) == name and _grid(d) == grid]
            return sum(v) / len(v) if v else float("nan")
        r_b, w_b = mean("FETCH_SIZE"), mean("WRITE_SIZE")
        a = next((alg[k] for k in alg if k in name), None)
        if a is None or ("kv_append" in name and grid != big_append):
            algs, ratio = "--", "--"
        else:
            algs, ratio = f"{a[0]:.4e} ({a[1]})", f"{r_b / a[0]:.4f}"
        out.append(f"| `{name}` | {grid} | {len(us)} | {sum(us) / len(us):.2f} | {min(us):.2f} | "
                   f"{max(us):.2f} | {r_b:.4e} | {w_b:.4e} | {algs} | {ratio} |")
    out += ["",
            "bench.py's HIP events around the whole calls of the same run (under the profiler): "
            f"append {det['t_kv_append_us (gamma+1 tokens, paged)']:.2f} us, greedy accept "
            f"{det['t_greedy_accept_us (fp32 logits, vocab 128256)']:.2f} us (both passes), "
            f"commit {det['t_kv_commit_us (lengths + 1024-slot ring)']:.2f} us.",
            "",
            f"Reading: the argmax pass streams the logits at {argmax_gbs:.0f} GB/s by kernel "
            "time; the appends,",
            "the acceptance pass and the commit are launch-latency bound (a few us each from a",
            "cold cache)."]
    return "\n".join(out) + "\n"


def summarize_lds(csv_path, bench_json, cmd):
    """LDS counters per kernel instance (means per dispatch over every dispatch
    of that instance in the run), the bench's timed verify and draft named."""
    rec = _bench_line(bench_json)
    W, K, S0 = rec["warmup"], rec["steps"], settle_count(rec)
    ds = _dispatches(_rows(csv_path))
    ver, dra = timed_calls(ds, W, K, S0)
    role = {ver[0][0]["name"]: "verify (bench)", dra[0][0]["name"]: "draft (bench)"}
    groups = {}
    for d in ds:
        if not d.get("SQ_LDS_IDX_ACTIVE") or "bench_" in d["name"]:
            continue  # kernels without LDS traffic (copies, fills) and the bench helpers
        groups.setdefault(d["name"], []).append(d)
    out = ["# LDS counters of the bench's kernels (rocprofv3 --pmc)",
           "",
           f"Workload: {WORKLOAD} (Llama-3.1-8B layer shape, B = 64, S = 32768, 16-token pages,",
           "gamma = 4) and the extra calls the bench times on it (one-token calls, the listed",
           "draft, SnapKV at prefill, the speculative-step kernels).  One MI355X (gfx950).",
           "Means per dispatch over every dispatch of each kernel instance, summed over the",
           "device as rocprofv3 reports them.",
           "",
           "Command (from /tmp with TMPDIR=/tmp; R = the repository root):",
           "",
           f"    {cmd}",
           "",
           "| kernel | dispatches | SQ_INSTS_LDS | SQ_LDS_IDX_ACTIVE (cycles) | SQ_LDS_BANK_CONFLICT (cycles) | conflict / active | SQ_LDS_ADDR_CONFLICT | SQ_LDS_UNALIGNED_STALL |",
           "|---|---|---|---|---|---|---|---|"]
    for name, dl in sorted(groups.items(), key=lambda kv: -sum(d.get("SQ_LDS_IDX_ACTIVE", 0) for d in kv[1])):
        m = {c: sum(d.get(c, 0.0) for d in dl) / len(dl) for c in LDS_COUNTERS}
        ratio = m["SQ_LDS_BANK_CONFLICT"] / m["SQ_LDS_IDX_ACTIVE"] if m["SQ_LDS_IDX_ACTIVE"] else 0.0
        label = (role[name] + " " if name in role else "") + f"`{_short(name)}`"
        out.append(f"| {label} | {len(dl)} | {m['SQ_INSTS_LDS']:.4g} | {m['SQ_LDS_IDX_ACTIVE']:.4g} | "
                   f"{m['SQ_LDS_BANK_CONFLICT']:.4g} | {ratio:.3f} | {m['SQ_LDS_ADDR_CONFLICT']:.4g} | "
                   f"{m['SQ_LDS_UNALIGNED_STALL']:.4g} |")
    snap = os.path.join(ROOT, "paper_2408_11049_amd", "csrc", "snapkv.hip")
    out += ["", f"kernel_source_sha256: {kernel_source_sha256()}",
            f"snapkv_source_sha256: {kernel_source_sha256([snap])}"]
    return "\n".join(out) + "\n"


ISSUE_COUNTERS = ["SQ_WAVES", "SQ_WAVE_CYCLES", "SQ_WAIT_ANY", "SQ_WAIT_INST_ANY",
                  "SQ_ACTIVE_INST_VALU", "SQ_INSTS_VALU", "SQ_INSTS_VALU_TRANS_F32",
                  "SQ_BUSY_CYCLES", "GRBM_GUI_ACTIVE"]


def summarize_issue(csv_path, bench_json, cmd, num_cus=256, num_xcds=8):
    """Where the waves of the SnapKV passes (and, for reference, the bench's
    verify and draft) spend their time: wave-cycles waiting for anything
    (a dependency: memory, LDS, a barrier) against waiting to issue (a ready
    instruction held back by a busy unit), the VALU busy fraction, VALU and
    transcendental instructions per wave and the clock, from one --pmc pass over
    a bench run.  GRBM_GUI_ACTIVE arrives summed over the XCDs."""
    rec = _bench_line(bench_json)
    W, K, S0 = rec["warmup"], rec["steps"], settle_count(rec)
    ds = _dispatches(_rows(csv_path))
    ver, dra = timed_calls(ds, W, K, S0)
    role = {ver[0][0]["name"]: "verify (bench)", dra[0][0]["name"]: "draft (bench)"}
    groups = {}
    for d in ds:
        if d["name"] in role or "snapkv_pass_kernel" in d["name"]:
            groups.setdefault(d["name"], []).append(d)
    out = ["# Issue and wait counters of the SnapKV passes (rocprofv3 --pmc)",
           "",
           f"Workload: the prompts of {WORKLOAD} (B = 64 prompts of 32768 tokens, Llama-3.1-8B",
           "heads, 16-token pages, 32 observation queries: 128 rows per kv head); the bench's",
           "verify and draft for reference.  One MI355X (gfx950).  Means per dispatch over every",
           "dispatch of each kernel instance.",
           "",
           "Command (from /tmp with TMPDIR=/tmp; R = the repository root):",
           "",
           f"    {cmd}",
           "",
           "wait (any) = SQ_WAIT_ANY / SQ_WAVE_CYCLES: the share of wave time spent waiting on",
           "a dependency (memory, LDS, a barrier); wait (issue) = SQ_WAIT_INST_ANY /",
           "SQ_WAVE_CYCLES: the share spent with an instruction ready but not issued (a busy",
           f"unit); cycles = GRBM_GUI_ACTIVE / {num_xcds} (it is reported summed over the XCDs); VALU",
           "busy = 100 x SQ_ACTIVE_INST_VALU / CUs / cycles (SQ_ACTIVE_INST_VALU counts quad-",
           "cycles of four SIMDs); clock = cycles / the dispatch's duration under the profiler.",
           "",
           "| kernel | dispatches | waves | wait (any) | wait (issue) | VALU busy % | VALU insts / wave | transcendental / wave | clock GHz |",
           "|---|---|---|---|---|---|---|---|---|"]
    for name, dl in sorted(groups.items(), key=lambda kv: -sum(d.get("SQ_WAVE_CYCLES", 0) for d in kv[1])):
        m = {c: sum(d.get(c, 0.0) for d in dl) / len(dl) for c in ISSUE_COUNTERS}
        cycles = m["GRBM_GUI_ACTIVE"] / num_xcds or 1.0
        ns = sum(d["end"] - d["start"] for d in dl) / len(dl)
        wc = m["SQ_WAVE_CYCLES"] or 1.0
        waves = m["SQ_WAVES"] or 1.0
        busy = 100.0 * m["SQ_ACTIVE_INST_VALU"] / num_cus / cycles
        label = (role[name] + " " if name in role else "") + f"`{_short(name)}`"
        out.append(f"| {label} | {len(dl)} | {m['SQ_WAVES']:.0f} | {m['SQ_WAIT_ANY'] / wc:.3f} | "
                   f"{m['SQ_WAIT_INST_ANY'] / wc:.3f} | {busy:.1f} | {m['SQ_INSTS_VALU'] / waves:.0f} | "
                   f"{m['SQ_INSTS_VALU_TRANS_F32'] / waves:.0f} | {cycles / ns:.2f} |")
    snap = os.path.join(ROOT, "paper_2408_11049_amd", "csrc", "snapkv.hip")
    out += ["", f"kernel_source_sha256: {kernel_source_sha256()}",
            f"snapkv_source_sha256: {kernel_source_sha256([snap])}"]
    return "\n".join(out) + "\n"


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-configs", action="store_true",
                    help="skip the per-configuration table (profiling passes)")
    ap.add_argument("--latency", action="store_true",
                    help="only the draft-call latency breakdown (profiles/)")
    ap.add_argument("--paged-ab", action="store_true",
                    help="only the paged / sequential-page / contiguous verify A/B (profiles/)")
    ap.add_argument("--summarize", choices=["trace", "counters", "mfma", "latency", "paged", "lds",
                                            "configs", "config-counters", "prefill", "steps",
                                            "issue"])
    ap.add_argument("--csv", nargs="+")
    ap.add_argument("--bench-json", nargs="+")
    ap.add_argument("--cmd", default="")
    args = ap.parse_args()
    if args.summarize:
        fn = {"trace": lambda: summarize_trace(args.csv[0], args.bench_json[0], args.cmd),
              "counters": lambda: summarize_counters(args.csv[0], args.csv[1], args.bench_json[0],
                                                     args.cmd),
              "mfma": lambda: summarize_mfma(args.csv[0], args.bench_json[0], args.cmd),
              "latency": lambda: summarize_latency(args.csv[0], args.bench_json[0], args.cmd),
              "paged": lambda: summarize_paged(args.csv[0], args.bench_json[0], args.cmd),
              "lds": lambda: summarize_lds(args.csv[0], args.bench_json[0], args.cmd),
              "issue": lambda: summarize_issue(args.csv[0], args.bench_json[0], args.cmd),
              "configs": lambda: summarize_configs(args.csv[0], args.bench_json[0], args.cmd),
              "config-counters": lambda: summarize_config_counters(
                  args.csv[0], args.csv[1], args.bench_json[0], args.bench_json[-1], args.cmd),
              "prefill": lambda: summarize_prefill(args.csv[0], args.csv[1], args.csv[2],
                                                   args.bench_json[0], args.cmd),
              "steps": lambda: summarize_steps(args.csv[0], args.csv[1], args.csv[2],
                                               args.bench_json[0], args.cmd)}
        sys.stdout.write(fn[args.summarize]())
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (the library has no multi-GPU path); "
              f"--gpus {args.gpus} is not supported", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2408_11049_amd as md
    from paper_2408_11049_amd import workloads as wl

    if not os.path.exists(md.LIB_PATH):
        raise SystemExit("libmagicdec.so is not built: run __graft_entry__.build() first")
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    if args.latency:
        print(json.dumps({"latency": latency_breakdown(dev)}), flush=True)
        return
    if args.paged_ab:
        print(json.dumps({"paged_ab": paged_ab(dev)}), flush=True)
        return
    w = wl.WORKLOADS[WORKLOAD]
    log(f"[bench] generating {WORKLOAD} on {torch.cuda.get_device_name(dev)}")
    c = wl.make_workload(w, device=dev)
    inputs = input_sha256(c)
    lens = c["kv_lens_np"]
    L = w.q_len
    out_v = torch.empty_like(c["q"])
    out_d = torch.empty_like(c["q"])
    lse_v = torch.empty(c["q"].shape[:3], dtype=torch.float32, device=dev)
    lse_d = torch.empty_like(lse_v)
    q1 = c["q"][:, :1].contiguous()
    out1 = torch.empty_like(q1)
    flush = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    lib = md.load_library()
    stream = torch.cuda.current_stream(dev)
    sh = md.ctypes.c_void_p(stream.cuda_stream)

    def ws(mode, q):
        n = md.md_workspace_bytes(q, c["k"], c["v"], c["kv_lens"], mode=mode, n_sink=w.n_sink,
                                  window=w.window, max_kv_len=c["max_kv_len"],
                                  page_table=c["page_table"])
        return torch.empty(max(n, 256), dtype=torch.uint8, device=dev) if n else None

    ws_v, ws_d, ws_v1, ws_d1 = ws(0, c["q"]), ws(1, c["q"]), ws(0, q1), ws(1, q1)

    common = dict(max_kv_len=c["max_kv_len"], page_table=c["page_table"])

    def verify():
        md.md_verify_attn(c["q"], c["k"], c["v"], c["kv_lens"], out=out_v, lse=lse_v,
                          workspace=ws_v, **common)

    def draft():
        md.md_draft_attn(c["q"], c["k"], c["v"], c["kv_lens"], w.n_sink, w.window, out=out_d,
                         lse=lse_d, workspace=ws_d, **common)

    def verify1():  # one query token per sequence: a plain decode step over the same cache
        md.md_verify_attn(q1, c["k"], c["v"], c["kv_lens"], out=out1, return_lse=False,
                          workspace=ws_v1, **common)

    def draft1():   # the real per-token draft step
        md.md_draft_attn(q1, c["k"], c["v"], c["kv_lens"], w.n_sink, w.window, out=out1,
                         return_lse=False, workspace=ws_d1, **common)

    flush_sink = torch.zeros(4, dtype=torch.float32, device=dev)

    def do_flush():
        # Cold cache: reading 1 GiB with cache-allocating loads evicts the L2s and
        # the 256 MB last-level cache, and leaves no dirty lines behind.
        md._check(lib.md_bench_evict(md.ctypes.c_void_p(flush.data_ptr()), flush.numel(),
                                     md.ctypes.c_void_p(flush_sink.data_ptr()), sh))

    def do_fill_flush():
        md._check(lib.md_bench_fill(md.ctypes.c_void_p(flush.data_ptr()), flush.numel(), 0, sh))

    bytes_v = kv_bytes(w, lens, "verify", L)
    bytes_d = kv_bytes(w, lens, "draft", L)

    # The host-side setup above (generation, hashing) leaves the GPU idle for
    # seconds: settle its clocks with SETTLE_CALLS untimed verify calls
    # (~100 ms) before the warm-up steps (see settle()).
    n_settle = settle(verify, do_flush, 0, torch.cuda.synchronize, min_calls=SETTLE_CALLS)
    log(f"[bench] settled with {n_settle} untimed verify calls; warmup {args.warmup} steps")
    for _ in range(args.warmup):
        do_flush(); verify()
        do_flush(); draft()
    torch.cuda.synchronize()

    K = args.steps
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(K)]
    log(f"[bench] timing {K} steps")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for s in range(K):
        do_flush()
        ev[s][0].record(stream); verify(); ev[s][1].record(stream)
        do_flush()
        ev[s][2].record(stream); draft(); ev[s][3].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    tv = np.array([e[0].elapsed_time(e[1]) for e in ev]) * 1e3  # us
    td = np.array([e[2].elapsed_time(e[3]) for e in ev]) * 1e3
    t_step_us = float(np.mean(tv + td))
    log(f"[bench] verify {np.median(tv):.1f} us  draft {np.median(td):.1f} us  (medians)")

    # Extra timings (outside the K-step region): the real one-token draft, the
    # one-token verify (KV-bound ratio the paper predicts ~1), the read ceiling.
    def timed(fn, n=10, flush_fn=None, stats=False):
        ts = []
        for _ in range(n):
            (flush_fn or do_flush)()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream); fn(); b.record(stream)
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b) * 1e3)
        if stats:
            return [round(float(x), 2) for x in np.percentile(ts, [10, 50, 90])]
        return float(np.median(ts))

    def timed_warm(fn, n=10):
        """Back-to-back calls, no flush: whatever of the cache the last call
        left in the L2s and the 256 MB last-level cache is reused."""
        fn()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        for _ in range(n):
            fn()
        b.record(stream)
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 1e3 / n

    t_verify_warm, t_draft_warm = timed_warm(verify), timed_warm(draft)
    # The same calls after a 1 GiB fill instead of a read (the dirty lines it
    # leaves are written back while the timed call runs).
    t_verify_fill, t_draft_fill = timed(verify, flush_fn=do_fill_flush), timed(draft, flush_fn=do_fill_flush)
    t_draft1 = timed(draft1)
    t_verify1 = timed(verify1)
    # SnapKV-style draft over a listed static cache at the paper's best SnapKV
    # budget (2049 positions per sequence and kv head, Sec. 5.2); seeded random
    # ascending prompt positions stand in for a selection.
    budget = 2049
    idx_np, n_np = wl.index_lists(w.B, w.Hkv, lens, L, budget, w.seed_base)
    idx_t = torch.from_numpy(idx_np).to(dev)
    n_t = torch.from_numpy(n_np).to(dev)

    def draft_idx():
        md.md_draft_attn_indexed(c["q"], c["k"], c["v"], c["kv_lens"], idx_t, n_t, out=out_d,
                                 return_lse=False, **common)

    t_draft_idx = timed(draft_idx)
    bytes_idx = int(sum((int(x) + L) for x in n_np)) * w.Hkv * 2 * w.d * w.esize

    # The steps around verification: append the gamma+1 tokens' K/V (new seeded
    # rows written over the cache's last L positions), greedy
    # acceptance over fp32 logits at the Llama-3 vocabulary, and the commit
    # with a rolling 1024-slot ring after the 2049-entry SnapKV-style lists.
    vocab = 128256
    k_new, v_new = wl.new_kv_rows(w.B, L, w.Hkv, w.d, w.dtype, seed=w.seed_base, device=dev)
    pos0 = (c["kv_lens"] - L).contiguous()
    lens_out = torch.empty_like(pos0)

    def append():
        md.md_kv_append(c["k"], c["v"], k_new, v_new, pos0, page_table=c["page_table"],
                        lens_out=lens_out)

    logits, draft_tok, _, _ = wl.step_logits(w.B, w.gamma, vocab, "f32", seed=w.seed_base,
                                             device=dev)
    acc = torch.empty((w.B,), dtype=torch.int32, device=dev)
    toks = torch.empty((w.B, L), dtype=torch.int32, device=dev)
    ws_acc = torch.empty((lib.md_greedy_accept_workspace_bytes(w.B, w.gamma, vocab),),
                         dtype=torch.uint8, device=dev)

    def accept():
        md.md_greedy_accept(logits, draft_tok, accepted=acc, tokens=toks, want_target=False,
                            workspace=ws_acc)

    ring = 1024
    lists = torch.full((w.B, w.Hkv, budget + ring), -1, dtype=torch.int32, device=dev)
    lists[:, :, :budget] = idx_t
    commit_lens = torch.empty_like(pos0)

    def commit():
        md.md_kv_commit(commit_lens, acc, L, idx=lists, ring_start=budget, ring_len=ring)

    # SnapKV-style selection at prefill over the same 32k-token prompts: 32
    # observation queries (the prompt's last positions), pooling 5, budget 2049.
    n_obs = 32
    q_obs = torch.randn((w.B, n_obs, w.Hq, w.d), generator=wl._gen(w.seed_base * 10 + 9, dev),
                        device=dev).to(torch.bfloat16)
    sk_kw = dict(max_prompt_len=c["max_kv_len"], page_table=c["page_table"])
    votes = md.md_snapkv_votes(q_obs, c["k"], c["kv_lens"], **sk_kw)
    ws_sk = torch.empty((max(md.md_snapkv_workspace_bytes(q_obs, c["k"], c["kv_lens"], **sk_kw), 256),),
                        dtype=torch.uint8, device=dev)
    sel_idx = torch.empty((w.B, w.Hkv, budget), dtype=torch.int32, device=dev)
    sel_len = torch.empty((w.B,), dtype=torch.int32, device=dev)
    t_votes = timed(lambda: md.md_snapkv_votes(q_obs, c["k"], c["kv_lens"], votes=votes,
                                               workspace=ws_sk, **sk_kw), n=5)
    t_select = timed(lambda: md.md_snapkv_select(votes, c["kv_lens"], n_obs, budget, pool=5,
                                                 idx=sel_idx, idx_len=sel_len), n=5)
    bytes_votes = 2 * int(sum(int(x) for x in lens)) * w.Hkv * w.d * w.esize  # K read twice

    t_append = timed(append)
    t_accept = timed(accept)
    ts = []
    for _ in range(10):
        commit_lens.copy_(pos0)
        do_flush()
        a_ev, b_ev = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a_ev.record(stream); commit(); b_ev.record(stream)
        torch.cuda.synchronize()
        ts.append(a_ev.elapsed_time(b_ev) * 1e3)
    t_commit = float(np.median(ts))
    bytes_append = 2 * 2 * w.B * L * w.Hkv * w.d * w.esize  # K and V rows, read + write

    # A whole speculative step as an engine issues it: gamma draft steps (one
    # token's K/V appended, then a one-token draft over the 2049-position
    # lists plus the 1024-slot ring), then the gamma+1 verified tokens' K/V,
    # verification, greedy acceptance and the commit.  Timed from the same
    # restored state each time, eagerly and as one HIP graph replay.
    sd_lists0 = torch.full((w.B, w.Hkv, budget + ring), -1, dtype=torch.int32, device=dev)
    sd_lists0[:, :, :budget] = idx_t
    sd_lists = sd_lists0.clone()
    sd_len = torch.full((w.B,), budget + ring, dtype=torch.int32, device=dev)
    sd_lens = pos0.clone()
    pos_i = [(pos0 + i).contiguous() for i in range(w.gamma)]
    kvl_i = [torch.empty_like(pos0) for _ in range(w.gamma)]
    k1 = [k_new[:, i:i + 1].contiguous() for i in range(w.gamma)]
    v1 = [v_new[:, i:i + 1].contiguous() for i in range(w.gamma)]
    out_sd1 = torch.empty_like(q1)
    ws_i1 = torch.empty((max(int(lib.md_workspace_bytes_indexed(md.ctypes.byref(md.make_args(
        q1, c["k"], c["v"], c["kv_lens"], **common)), budget + ring)), 256),), dtype=torch.uint8,
        device=dev)
    ws_vsd = ws(0, c["q"])
    sd_out = torch.empty_like(pos0)

    def sd_step():
        for i in range(w.gamma):
            md.md_kv_append(c["k"], c["v"], k1[i], v1[i], pos_i[i], page_table=c["page_table"],
                            lens_out=kvl_i[i])
            md.md_draft_attn_indexed(q1, c["k"], c["v"], kvl_i[i], sd_lists, sd_len, out=out_sd1,
                                     return_lse=False, workspace=ws_i1, **common)
        md.md_kv_append(c["k"], c["v"], k_new, v_new, sd_lens, page_table=c["page_table"],
                        lens_out=sd_out)
        md.md_verify_attn(c["q"], c["k"], c["v"], sd_out, out=out_v, lse=lse_v, workspace=ws_vsd,
                          **common)
        md.md_greedy_accept(logits, draft_tok, accepted=acc, tokens=toks, want_target=False,
                            workspace=ws_acc)
        md.md_kv_commit(sd_lens, acc, L, idx=sd_lists, ring_start=budget, ring_len=ring)

    def sd_timed_pair(eager, replay, restore, n=12):
        """Median step time eagerly and as a graph replay, the two forms
        alternating (each from the same restored state, after an eviction),
        so drift over the run affects both alike."""
        ts = ([], [])
        for _ in range(n):
            for j, run in enumerate((eager, replay)):
                restore()
                do_flush()
                a_ev, b_ev = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a_ev.record(stream); run(); b_ev.record(stream)
                torch.cuda.synchronize()
                ts[j].append(a_ev.elapsed_time(b_ev) * 1e3)
        return float(np.median(ts[0])), float(np.median(ts[1]))

    def sd_restore():
        sd_lens.copy_(pos0)
        sd_lists.copy_(sd_lists0)

    sd_step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            sd_step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    t_sd_eager, t_sd_graph = sd_timed_pair(sd_step, graph.replay, sd_restore)

    # The same selection gathered once into a draft cache of its own
    # (md_kv_gather): a draft step is then verify attention over the 2049
    # gathered rows plus its own speculated rows, appended to that cache.
    cap_c = budget + L + w.gamma
    ck = torch.empty((w.B, cap_c, w.Hkv, w.d), dtype=c["k"].dtype, device=dev)
    cv = torch.empty_like(ck)
    glen = torch.empty_like(pos0)

    def gather():
        md.md_kv_gather(ck, cv, c["k"], c["v"], idx_t, n_t, pos0, dst_lens=glen,
                        src_page_table=c["page_table"])

    t_gather = timed(gather, n=5)
    gather()
    torch.cuda.synchronize()
    common_c = dict(max_kv_len=cap_c)
    glen1, glenL = (glen + 1).contiguous(), (glen + L).contiguous()

    def ws_c(q, lens_c):
        n = md.md_workspace_bytes(q, ck, cv, lens_c, mode=md.MD_MODE_VERIFY, **common_c)
        return torch.empty((max(n, 256),), dtype=torch.uint8, device=dev) if n else None

    ws_g1, ws_gL = ws_c(q1, glen1), ws_c(c["q"], glenL)
    t_draft_g1 = timed(lambda: md.md_verify_attn(q1, ck, cv, glen1, out=out_sd1, return_lse=False,
                                                 workspace=ws_g1, **common_c))
    t_draft_gL = timed(lambda: md.md_verify_attn(c["q"], ck, cv, glenL, out=out_d,
                                                 return_lse=False, workspace=ws_gL, **common_c))
    g_lens = glen.clone()
    g_pos_i = [(glen + i).contiguous() for i in range(w.gamma)]
    g_kvl_i = [torch.empty_like(pos0) for _ in range(w.gamma)]
    g_out = torch.empty_like(pos0)

    def sd_step_gathered():
        for i in range(w.gamma):
            md.md_kv_append(ck, cv, k1[i], v1[i], g_pos_i[i], lens_out=g_kvl_i[i])
            md.md_verify_attn(q1, ck, cv, g_kvl_i[i], out=out_sd1, return_lse=False,
                              workspace=ws_g1, **common_c)
        md.md_kv_append(c["k"], c["v"], k_new, v_new, sd_lens, page_table=c["page_table"],
                        lens_out=sd_out)
        md.md_kv_append(ck, cv, k_new, v_new, g_lens, lens_out=g_out)
        md.md_verify_attn(c["q"], c["k"], c["v"], sd_out, out=out_v, lse=lse_v, workspace=ws_vsd,
                          **common)
        md.md_greedy_accept(logits, draft_tok, accepted=acc, tokens=toks, want_target=False,
                            workspace=ws_acc)
        md.md_kv_commit(sd_lens, acc, L)
        md.md_kv_commit(g_lens, acc, L)

    def sdg_restore():
        sd_lens.copy_(pos0)
        g_lens.copy_(glen)

    sd_step_gathered()
    torch.cuda.synchronize()
    graph_g = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph_g, stream=side):
            sd_step_gathered()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    t_sdg_eager, t_sdg_graph = sd_timed_pair(sd_step_gathered, graph_g.replay, sdg_restore)
    bytes_gather = 2 * bytes_idx - 2 * w.B * L * w.Hkv * 2 * w.d * w.esize  # rows read + written
    bytes_logits = logits.numel() * logits.element_size()
    # A plain 1 GiB copy of known size: its FETCH_SIZE / WRITE_SIZE readings
    # calibrate the HBM byte counters of a rocprofv3 --pmc run of this script.
    md._check(lib.md_bench_copy(md.ctypes.c_void_p(flush.data_ptr()),
                                md.ctypes.c_void_p(c["k"].data_ptr()), flush.numel(), sh))
    sink = torch.zeros(4, dtype=torch.float32, device=dev)
    kbytes = c["k"].numel() * c["k"].element_size()
    t_read = timed(lambda: md._check(lib.md_bench_stream_read(
        md.ctypes.c_void_p(c["k"].data_ptr()), kbytes, md.ctypes.c_void_p(sink.data_ptr()), sh)))
    ceiling = kbytes / (t_read * 1e-6) / 1e9
    torch.cuda.synchronize()

    verify_gbs = bytes_v / (np.mean(tv) * 1e-6) / 1e9
    value = (bytes_v + bytes_d) / (t_step_us * 1e-6) / 1e9
    traffic = read_counters()
    trace = read_trace()
    mfma = read_mfma()
    kernel_time = None
    if trace:
        kernel_time = {
            "mean_us": trace["verify_kernel_mean_us"],
            "achieved": round(bytes_v / (trace["verify_kernel_mean_us"] * 1e-6) / 1e9, 1),
            "frac": round(bytes_v / (trace["verify_kernel_mean_us"] * 1e-6) / 1e9 / HBM_PEAK_GBS, 4),
            "event_mean_us_same_run": trace["verify_event_mean_us"],
            "source": os.path.relpath(PROFILE_TRACE, ROOT) + " (the timed dispatches of a traced run)"}
    roofline = {"bound": "hbm", "achieved": round(verify_gbs, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(verify_gbs / HBM_PEAK_GBS, 4),
                "traffic": traffic,
                "kernel": "md::attn_partial_kernel (md_verify_attn), a single launch",
                "algorithmic_bytes_per_launch": bytes_v,
                "kernel_time": kernel_time,
                "mfma": mfma}
    configs = None
    if not args.no_configs:
        configs = config_table(CONFIGS, dev, timed,
                               settle_fn=lambda fn: settle(fn, do_flush, 60, torch.cuda.synchronize))
        configs[WORKLOAD + " (headline: the event means above)"] = {
            "t_verify_us_p10_p50_p90": [round(float(x), 2) for x in np.percentile(tv, [10, 50, 90])],
            "t_verify_qlen1_us": round(t_verify1, 2),
            "t_verify_us_after_fill (1 GiB written before each call, not read)": round(t_verify_fill, 2),
            "t_draft_us_after_fill": round(t_draft_fill, 2),
            "t_draft_us_p10_p50_p90": [round(float(x), 2) for x in np.percentile(td, [10, 50, 90])],
            "t_draft_qlen1_us": round(t_draft1, 2),
            "verify_frac": round(bytes_v / (np.median(tv) * 1e-6) / 1e9 / HBM_PEAK_GBS, 4),
            "draft_frac": round(bytes_d / (np.median(td) * 1e-6) / 1e9 / HBM_PEAK_GBS, 4),
            "draft_qlen1_frac": round(kv_bytes(w, lens, "draft", 1) / (t_draft1 * 1e-6) / 1e9 / HBM_PEAK_GBS, 4),
            "t_sd_us (gamma x draft_qlen1 + verify)": round(w.gamma * t_draft1 + float(np.median(tv)), 2),
            "verify_ratio_qlen_gamma1_vs_1": round(float(np.median(tv)) / t_verify1, 4)}

    cpu = None
    oracle_extras = None
    if not args.no_cpu_baseline:
        log("[bench] cpu baseline (fp64 oracle on a bounded sample)")
        cpu = cpu_baseline(c, w)
        oracle_extras = cpu_oracle_extras(c, w, logits, draft_tok, q_obs, n_obs, t_accept, t_votes)

    rec = {
        "metric": "K/V HBM GB/s (% of peak) and µs per verify+draft attention step",
        "value": round(value, 1), "unit": "GB/s", "n_gpus": 1, "steps": K,
        "warmup": args.warmup, "ms_per_step": round(t_step_us / 1e3, 5),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": WORKLOAD, "B": w.B, "Hq": w.Hq, "Hkv": w.Hkv, "head_dim": w.d,
                   "S": w.S, "gamma": w.gamma, "n_sink": w.n_sink, "window": w.window,
                   "page_size": w.page_size,
                   "cache": "cold (a 1 GiB read evicts the caches before each call)"},
        "roofline": roofline,
        "cpu_baseline": cpu,
        "inputs_sha256": inputs,
        "detail": {
            "pct_of_hbm_peak": round(100 * value / HBM_PEAK_GBS, 2),
            "settle_calls (untimed verify calls before the warm-up)": n_settle,
            "t_verify_us": round(float(np.mean(tv)), 2),
            "t_verify_us_p10_p50_p90": [round(float(x), 2) for x in np.percentile(tv, [10, 50, 90])],
            "t_draft_us": round(float(np.mean(td)), 2),
            "t_draft_us_p10_p50_p90": [round(float(x), 2) for x in np.percentile(td, [10, 50, 90])],
            "t_draft_qlen1_us": round(t_draft1, 2),
            "t_verify_warm_us (back-to-back, no flush)": round(t_verify_warm, 2),
            "t_draft_warm_us (back-to-back, no flush)": round(t_draft_warm, 2),
            "t_verify_qlen1_us": round(t_verify1, 2),
            "t_verify_us_after_fill (1 GiB written before each call, not read)": round(t_verify_fill, 2),
            "t_draft_us_after_fill": round(t_draft_fill, 2),
            "verify_ratio_qlen_gamma1_vs_1": round(float(np.median(tv)) / t_verify1, 4),
            "t_sd_us (gamma*t_draft(1) + t_verify)": round(w.gamma * t_draft1 + float(np.mean(tv)), 2),
            "t_draft_indexed_us (SnapKV-style list, budget 2049)": round(t_draft_idx, 2),
            "draft_indexed_kv_bytes": bytes_idx,
            "draft_indexed_gbs": round(bytes_idx / (t_draft_idx * 1e-6) / 1e9, 1),
            "t_snapkv_votes_us (prefill, 32 observation queries)": round(t_votes, 2),
            "snapkv_votes_k_bytes (two passes over K)": bytes_votes,
            "snapkv_votes_gbs": round(bytes_votes / (t_votes * 1e-6) / 1e9, 1),
            "t_snapkv_select_us (pool 5, budget 2049)": round(t_select, 2),
            "t_kv_append_us (gamma+1 tokens, paged)": round(t_append, 2),
            "kv_append_bytes (read + write)": bytes_append,
            "t_greedy_accept_us (fp32 logits, vocab 128256)": round(t_accept, 2),
            "greedy_accept_logits_bytes": bytes_logits,
            "greedy_accept_gbs": round(bytes_logits / (t_accept * 1e-6) / 1e9, 1),
            "t_kv_commit_us (lengths + 1024-slot ring)": round(t_commit, 2),
            "t_sd_full_us (gamma*t_draft(1) + append + verify + accept + commit)": round(
                w.gamma * t_draft1 + t_append + float(np.mean(tv)) + t_accept + t_commit, 2),
            "t_sd_step_eager_us (gamma x (append 1 + listed draft 1) + append + verify + accept + commit)":
                round(t_sd_eager, 2),
            "t_sd_step_graph_us (the same step, one HIP graph replay; the two forms alternate)":
                round(t_sd_graph, 2),
            "t_kv_gather_us (the 2049 listed rows into a draft cache, once per prompt)":
                round(t_gather, 2),
            "kv_gather_bytes (read + write)": bytes_gather,
            "t_draft_gathered_qlen1_us (verify over the gathered 2049 rows + 1)": round(t_draft_g1, 2),
            "t_draft_gathered_us (q_len gamma+1)": round(t_draft_gL, 2),
            "draft_gathered_gbs": round(bytes_idx / (t_draft_gL * 1e-6) / 1e9, 1),
            "t_sd_step_gathered_eager_us (the step with drafts over the gathered cache)":
                round(t_sdg_eager, 2),
            "t_sd_step_gathered_graph_us": round(t_sdg_graph, 2),
            "verify_kv_bytes": bytes_v, "draft_kv_bytes": bytes_d,
            "verify_gbs": round(verify_gbs, 1),
            "draft_gbs": round(bytes_d / (np.mean(td) * 1e-6) / 1e9, 1),
            "read_ceiling_gbs": round(ceiling, 1),
            "pct_of_read_ceiling": round(100 * value / ceiling, 2),
            "wall_ms_per_step_incl_flush": round(wall * 1e3 / K, 4),
            "configs": configs,
            "cpu_oracle_extras": oracle_extras,
            "paper_context": "2.51x end-to-end speedup, Llama-3.1-8B SnapKV self-speculation, "
                             "8xH100 (Table 2): context only, not comparable",
        },
    }
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
