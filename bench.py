"""Benchmark of one draft + verify step on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]
    python bench.py --copy-probe BYTES      (counter calibration only, see profiles/)

A step = spec_draft followed by spec_verify, enqueued back to back on one
stream, on one batch of seeded synthetic inputs that are resident in HBM before
the timed region starts (the base model's forward between the two calls is not
part of this path; its logits are pre-generated).  Prints ONE JSON line.

The metric is quoted at batch 1 and at batch 64.  `value`, `config`, `roofline`
and `cpu_baseline` are those of the batch-1 workload (`llama7b_b1`, bound by HBM
bandwidth); with the default workload the line also carries a `batch64` object:
the same measurement of `llama7b_b64` (bound by the matrix cores), with its own
`roofline` for the dominant dense kernel and the fraction of the bf16 MFMA peak
the whole draft reaches.

Extra objects on the line:
  roofline      dominant contraction kernel: algorithmic bytes (or flops) per
                launch / its average launch duration, measured live with HIP
                events recorded by the library around each launch (on the
                stream the kernels run on), against the MI355X peak.
  cpu_baseline  the CPU oracle (as it stands) timed on the host cores on a
                bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X HBM3E, published
MFMA_BF16_PEAK_TFLOPS = 2500.0   # MI355X dense bf16, published
# labels of spec_launch_record_t.kernel: the kernel instances as rocprofv3 names them
def kernel_name(kid: int) -> str:
    if kid >= 1000:
        mb, rest = divmod(kid - 1000, 100)
        return "head_gemm32_kernel<%d, 2, %d, %s>" % (mb, rest // 2, "true" if rest % 2 else "false")
    if kid >= 400:
        nb, rest = (4, kid - 500) if kid >= 500 else (5, kid - 400)
        return "head_once_kernel<%d, %d, %d>" % ((nb,) + divmod(rest, 10))
    if kid >= 300:
        return "head_panel_kernel<%d, %d>" % divmod(kid - 300, 10)
    if kid >= 100:
        mb, kt = divmod(kid - 100, 20)
        return "head_tile_kernel<%d, %d>" % (mb, kt)
    return {0: "head_skinny_kernel", 1: "head_gemm_kernel<2, 1, 8>", 2: "head_skinny32_kernel"}[kid]


def kernel_sources_digest() -> str:
    """Digest of the library's kernel sources: a stored counter measurement belongs to the
    kernels it was taken on, and is dropped once they change."""
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2404_19124_amd", "csrc")
    for name in sorted(os.listdir(csrc)):
        with open(os.path.join(csrc, name), "rb") as f:
            h.update(name.encode() + b"\0" + f.read())
    return h.hexdigest()[:16]


def measure(wl_name: str, steps: int, warmup: int, verbose: bool = False):
    """Times `steps` whole steps of one workload, then the same number again with the library's
    per-launch events on, and the draft and the verify alone.  Returns (metrics dict, context for
    the CPU baseline)."""
    import torch
    from paper_2404_19124_amd import binding as B
    from paper_2404_19124_amd import workloads as W
    from paper_2404_19124_amd.runner import Step

    wl = W.WORKLOADS[wl_name]
    gen = W.make_generator(wl.seed, "cuda")
    w = W.make_speculator(wl, gen, device="cuda")
    state, last = W.make_draft_inputs(wl, gen, device="cuda")
    step = Step(wl, w)
    stream = torch.cuda.current_stream()

    # inputs of verify: logits boosted at the candidates this draft produces
    step.draft(state, last)
    torch.cuda.synchronize()
    logits = W.make_base_logits(wl, step.cand_tokens, gen, device="cuda")
    torch.cuda.synchronize()

    def one_step():
        step.draft(state, last, stream)
        step.verify(logits, None, stream)

    def timed(fn, reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        return time.perf_counter() - t0

    def settle(fn, reps):
        """Untimed passes of the loop that is about to be timed, until two in a row take the same time.
        On this stack the host-side enqueue goes through a one-time slow phase after the first ~2000
        launches of a process (a 200-step loop then takes twice its time, reproducibly the second such
        loop); that is the runtime's warm-up, not the path's, and a serving process is past it for good."""
        prev = timed(fn, reps)
        for _ in range(6):
            cur = timed(fn, reps)
            if abs(cur - prev) <= 0.03 * cur:
                break
            prev = cur

    for _ in range(warmup):
        one_step()
    settle(one_step, max(steps, 200))
    dt = timed(one_step, steps)
    ms_per_step = dt * 1e3 / steps
    steps_per_s = steps / dt
    mean_accept = float(step.accept_len.float().mean())
    # (each half alone)
    settle(lambda: step.draft(state, last, stream), steps)
    ms_draft = timed(lambda: step.draft(state, last, stream), steps) * 1e3 / steps
    settle(lambda: step.verify(logits, None, stream), steps)
    ms_verify = timed(lambda: step.verify(logits, None, stream), steps) * 1e3 / steps

    # ---- dominant kernel, timed live with events around each launch
    B.spec_profile_enable(step.model, 16 * steps)
    ms_per_step_events = timed(one_step, steps) * 1e3 / steps
    recs = B.spec_profile_read(step.model, 16 * steps)
    B.spec_profile_enable(step.model, 0)
    by_kernel = {}
    for r in recs:
        d = by_kernel.setdefault(r["kernel"], {"ms": 0.0, "n": 0, "bytes": 0.0, "flops": 0.0})
        d["ms"] += r["ms"]
        d["n"] += 1
        # algorithmic traffic of a launch: the weights once, the state rows once
        d["bytes"] += 2.0 * r["weight_rows"] * r["k"] + 2.0 * r["rows"] * r["k"]
        d["flops"] += 2.0 * r["rows"] * r["weight_rows"] * r["k"]
    if verbose:
        groups = {}
        for r in recs:
            g = groups.setdefault((r["kernel"], r["rows"], r["weight_rows"], r["k"]), [0.0, 0])
            g[0] += r["ms"]
            g[1] += 1
        for (kern, rows, wrows, kk), (ms, cnt) in sorted(groups.items()):
            us = ms / cnt * 1e3
            print("  %-24s rows %5d x weights %6d x k %5d : %8.2f us  %7.1f GB/s  %7.1f TFLOP/s  (%d launches)"
                  % (kernel_name(kern), rows, wrows, kk, us, (2.0 * wrows * kk + 2.0 * rows * kk) / us / 1e3,
                     2.0 * rows * wrows * kk / us / 1e6, cnt), file=sys.stderr)
    dom = max(by_kernel, key=lambda k: by_kernel[k]["ms"])
    d = by_kernel[dom]
    avg_ms = d["ms"] / d["n"]
    gbs = d["bytes"] / d["n"] / (avg_ms * 1e-3) / 1e9
    tflops = d["flops"] / d["n"] / (avg_ms * 1e-3) / 1e12
    # which roof binds this kernel: compare the two ideal times
    t_hbm = d["bytes"] / d["n"] / (HBM_PEAK_GBS * 1e9)
    t_mfma = d["flops"] / d["n"] / (MFMA_BF16_PEAK_TFLOPS * 1e12)
    traffic = _traffic_from_profiles(wl_name, kernel_name(dom))
    if t_hbm >= t_mfma:
        roofline = {"bound": "hbm", "achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": round(gbs / HBM_PEAK_GBS, 4), "traffic": traffic}
    else:
        roofline = {"bound": "mfma", "achieved": round(tflops, 1), "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                    "frac": round(tflops / MFMA_BF16_PEAK_TFLOPS, 4), "traffic": traffic}
    roofline.update({"kernel": kernel_name(dom), "avg_launch_us": round(avg_ms * 1e3, 2),
                     "launches_per_step": d["n"] / steps,
                     "algorithmic_bytes_per_launch": d["bytes"] / d["n"],
                     "flops_per_launch": d["flops"] / d["n"],
                     "gbs": round(gbs, 1), "tflops": round(tflops, 2),
                     "ms_per_step_with_events": round(ms_per_step_events, 4),
                     "share_of_step": round(d["ms"] / steps / ms_per_step_events, 3)})
    # all contraction launches of a step together (every head and projection)
    all_ms = sum(x["ms"] for x in by_kernel.values()) / steps
    all_flops = sum(x["flops"] for x in by_kernel.values()) / steps

    ab = wl.algorithmic_bytes()
    out = {
        "workload": wl.name, "value": round(steps_per_s, 2), "ms_per_step": round(ms_per_step, 5),
        "ms_draft": round(ms_draft, 5), "ms_verify": round(ms_verify, 5),
        "step_algorithmic_bytes": ab["total"],
        "step_hbm_gbs": round(ab["total"] / (ms_per_step * 1e-3) / 1e9, 1),
        "step_hbm_frac": round(ab["total"] / (ms_per_step * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
        "step_contraction_tflops": round(wl.contraction_flops() / (ms_per_step * 1e-3) / 1e12, 2),
        # the draft's heads and projections against the bf16 MFMA peak: over the draft's wall time, and over
        # the contraction launches alone (their event durations)
        "draft_mfma_frac": round(wl.contraction_flops() / (ms_draft * 1e-3) / 1e12 / MFMA_BF16_PEAK_TFLOPS, 4),
        "contractions_mfma_frac": round(all_flops / (all_ms * 1e-3) / 1e12 / MFMA_BF16_PEAK_TFLOPS, 4),
        "verify_hbm_frac": round(ab["base_logits"] / (ms_verify * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
        "mean_accept_len_synthetic": round(mean_accept, 3),
        "roofline": roofline,
    }
    return out, (wl, w, state, last, logits, step)


def config_of(wl) -> dict:
    return {"workload": wl.name, "batch": wl.batch, "emb_dim": wl.emb_dim, "inner_dim": wl.inner_dim,
            "vocab": wl.vocab, "n_predict": wl.n_predict, "top_k": list(wl.top_k), "B": wl.B,
            "logits_dtype": wl.logits_dtype, "seed": wl.seed}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="llama7b_b1")
    ap.add_argument("--no-batch64", action="store_true", help="leave out the batch-64 half of the metric")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=12.0)
    ap.add_argument("--verbose", action="store_true", help="per-shape timing of the contraction launches on stderr")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="BYTES",
                    help="instead of the benchmark: launch the library's plain copy kernel over BYTES a few times "
                         "(calibration of rocprofv3's FETCH_SIZE / WRITE_SIZE counters) and exit")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU; --gpus %d is not supported (no collectives, no sharding in "
              "this path)" % args.gpus, file=sys.stderr)
        return 2

    import torch
    from paper_2404_19124_amd import binding as B

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 2
    torch.cuda.set_device(0)
    if args.copy_probe:
        n = args.copy_probe // 16 * 16
        src = torch.full((n,), 3, dtype=torch.uint8, device="cuda")
        dst = torch.zeros(n, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        for _ in range(5):
            B.spec_copy_probe(src, dst, torch.cuda.current_stream())
        torch.cuda.synchronize()
        ok = bool(torch.equal(src, dst))
        print(json.dumps({"copy_probe_bytes": n, "launches": 5, "copied_correctly": ok}), flush=True)
        return 0 if ok else 1

    m, ctx = measure(args.workload, args.steps, args.warmup, args.verbose)
    wl = ctx[0]
    out = {
        "metric": "draft+verify steps/s", "value": m.pop("value"), "unit": "steps/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": m.pop("ms_per_step"),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": wl.weight_dtype, "data": "synthetic", "config": config_of(wl),
    }
    m.pop("workload")
    out.update(m)
    out["cpu_baseline"] = None if args.no_cpu_baseline else _cpu_baseline(*ctx, args.cpu_seconds)
    ctx[-1].close()
    del ctx
    torch.cuda.empty_cache()
    if args.workload == "llama7b_b1" and not args.no_batch64:
        # the batch-64 half of the metric: same protocol, the dense (MFMA) kernels
        m64, ctx64 = measure("llama7b_b64", args.steps, args.warmup, args.verbose)
        m64["unit"] = "steps/s"
        m64["steps"], m64["warmup"] = args.steps, args.warmup
        m64["config"] = config_of(ctx64[0])
        out["batch64"] = m64
        ctx64[-1].close()
    print(json.dumps(out), flush=True)
    return 0


def _traffic_from_profiles(workload: str, kernel: str):
    """HBM bytes per launch of the dominant kernel, measured with rocprofv3 --pmc
    (FETCH_SIZE, WRITE_SIZE) and kept as text under profiles/; None when no such
    measurement has been recorded for this workload and kernel instance, or when the
    kernel sources have changed since it was taken."""
    path = os.path.join(ROOT, "profiles", "hbm_traffic.json")
    try:
        with open(path) as f:
            table = json.load(f)
        entry = table.get(workload, {}).get(kernel)
        if not isinstance(entry, dict) or entry.get("kernel_sources") != kernel_sources_digest():
            return None
        return entry.get("bytes_per_launch")
    except (OSError, ValueError):
        return None


def _cpu_baseline(wl, w, state, last, logits, step, budget_s: float):
    """The oracle timed on the host: whole steps on a bounded number of sequences."""
    from oracle import spec_oracle as O
    from paper_2404_19124_amd import workloads as W

    try:
        cores = len(os.sched_getaffinity(0))
    except AttributeError:
        cores = os.cpu_count() or 1
    # numpy's BLAS does the oracle's matmuls: its pool size is the number of threads really used
    try:
        from threadpoolctl import threadpool_info
        threads = max([p.get("num_threads", 1) for p in threadpool_info()] + [1])
    except ImportError:
        threads = cores
    wn = W.weights_to_numpy(w)
    nseq = min(wl.batch, 2)
    st = W.to_numpy_f32(state[:nseq])
    lt = last[:nseq].cpu().numpy()
    lg = W.to_numpy_f32(logits[:nseq])
    cand = step.cand_tokens[:nseq].cpu().numpy()
    # one untimed call sizes the sample
    t0 = time.perf_counter()
    O.draft(wn, st[:1], lt[:1], wl.top_k, wl.B, state_dtype=wl.weight_dtype)
    O.verify(lg[:1], cand[:1])
    per_seq = time.perf_counter() - t0
    nseq = 1 if per_seq * 2 > budget_s or wl.batch == 1 else nseq
    reps = max(1, min(60, int(budget_s / max(per_seq * nseq, 1e-3))))
    t0 = time.perf_counter()
    for _ in range(reps):
        d = O.draft(wn, st[:nseq], lt[:nseq], wl.top_k, wl.B, state_dtype=wl.weight_dtype)
        O.verify(lg[:nseq], d.cand_tokens)
    dt = (time.perf_counter() - t0) / reps
    # a step covers the whole batch: scale the sampled sequences up (sequences are independent)
    step_s = dt * wl.batch / nseq
    return {"value": round(1.0 / step_s, 4), "unit": "steps/s", "cores": min(threads, cores), "kind": "oracle",
            "host_cores": cores,
            "sample": "%d whole draft+verify step(s) of %d of %d sequence(s), %d repetition(s), %.2f s each; "
                      "scaled by batch/sample" % (reps, nseq, wl.batch, reps, dt)}


if __name__ == "__main__":
    sys.exit(main())
