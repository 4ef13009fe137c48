"""Benchmark of the hot path on one MI355X.

One "step" = one pass of the whole path over one synthetic batch: fused causal
prefill attention + observation-window importance, then top-k selection with
index compaction.  Inputs are resident in HBM before the timed region.

Prints ONE JSON line (see the field notes at the bottom of this file).  The
top-level fields are those of the 32k-token prompt (the configuration the
target is quoted on); `configs` carries the same measurements for the other
four configurations.  Every configuration is also compared with the CPU
oracle on the same tensors in the same run (`parity`); a mismatch makes the
benchmark exit with status 1.
"""
import argparse
import ctypes
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0      # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0
HEADLINE = "c4"
OTHERS = ("c1", "c2", "c3", "c5")

# HBM bytes per launch of the attention kernel (FETCH_SIZE + WRITE_SIZE of rocprofv3 --pmc runs, each
# scaled by the same counter's reading for a 1 GiB device copy; see profiles/).  Valid only for the
# kernel sources with this digest: once they change the figure is reported as null.
KERNEL_SOURCES = ("attn_fwd.hpp", "attn_wide.hpp")
TRAFFIC = {"c4": {"bytes": 1.688e9, "sources_sha256": "afa03a21771c1c55c95d8d70c4d43d1a2e3ad540c9291b9d44990b12f0edd02d"}}

O_ATOL, REL = 2e-2, 1e-3       # the parity bar: O max-abs, log-sum-exp / importance relative


def kernel_digest():
    """Digest of the attention kernel's code: its sources without // comments and white space, so
    that the stored traffic figure survives a reworded comment and nothing else."""
    import hashlib
    import re
    h = hashlib.sha256()
    for name in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2508_09035_amd", "csrc", name), "r", encoding="utf-8") as f:
            code = re.sub(r"//[^\n]*", "", f.read())
        h.update(re.sub(r"\s+", "", code).encode())
    return h.hexdigest()


def time_gpu(fn, iters, warmup, prewarm_ms=100.0):
    """Average milliseconds per call between two HIP events on the stream the calls are enqueued on.
    Before the `warmup` untimed calls the same call is repeated for about `prewarm_ms` of GPU time
    (untimed as well): after the seconds of host work that precede a measurement (oracle, uploads)
    the GPU sits at its idle clocks and needs some milliseconds of work to leave them, which a
    handful of sub-millisecond warm-up calls is not (the 0.4 ms step of the chunked configuration
    measured 13 % slow that way)."""
    import torch
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(3):
        fn()
    stop.record()
    torch.cuda.synchronize()
    per_call = max(start.elapsed_time(stop) / 3, 1e-3)
    for _ in range(min(5000, int(prewarm_ms / per_call))):
        fn()
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(iters):
        fn()
    stop.record()
    torch.cuda.synchronize()
    return start.elapsed_time(stop) / iters


def time_gpu_each(fn, iters):
    """Median and minimum milliseconds of single calls (one HIP event pair per call, GPU already warm)."""
    import torch
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(iters)]
    for a, b in evs:
        a.record()
        fn()
        b.record()
    torch.cuda.synchronize()
    ms = sorted(a.elapsed_time(b) for a, b in evs)
    return ms[len(ms) // 2], ms[0]


def oracle_sample(wl, budget_gflop):
    """The oracle (as it stands) on a bounded seeded sample of query rows of the workload, timed on
    the host cores.  Returns the rows, its O and log-sum-exp for them, the flops and the seconds."""
    import numpy as np
    import oracle
    d, hq = wl.head_dim, wl.n_q_heads
    rng = np.random.default_rng(1234)
    rows, flops = [], 0.0
    cu_q, cu_k = wl.cu_seqlens_q, wl.cu_seqlens_k
    for r in rng.permutation(wl.total_q):
        b = int(np.searchsorted(cu_q, r, side="right") - 1)
        i = int(r - cu_q[b])
        n_vis = i + int((cu_k[b + 1] - cu_k[b]) - (cu_q[b + 1] - cu_q[b])) + 1
        rows.append(int(r))
        flops += 4.0 * d * hq * n_vis
        if flops >= budget_gflop * 1e9:
            break
    rows = np.array(sorted(rows), dtype=np.int32)
    t0 = time.perf_counter()
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, cu_q, cu_k, wl.scale, rows=rows)
    return rows, oO, oL, flops, time.perf_counter() - t0


def parity(wl, dev, rows, oO, oL):
    """The outputs of one step against the oracle: O and log-sum-exp on the sampled rows,
    importance and the selected index sets in full (indices may differ only where the oracle's
    score lies within the score tolerance of the k-th score)."""
    import numpy as np
    import oracle
    dev.poison()
    dev.step()
    O, lse, imp, idx, mask = dev.results()
    o_err = float(np.abs(O[rows] - oO).max()) if len(rows) else 0.0
    l_rel = float((np.abs(lse[:, rows] - oL) / np.maximum(np.abs(oL), 1e-6)).max()) if len(rows) else 0.0
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale,
                           -1 if wl.chunked else wl.window)
    i_rel = float((np.abs(imp - oI) / np.maximum(np.abs(oI), 1e-6)).max())
    want_idx, want_mask = oracle.select_topk(oI, wl.cu_seqlens_k, wl.k_keep, wl.cand_begin, wl.cand_end)
    cu_keep = wl.cu_keep
    beyond_ties = tie_swaps = 0
    for g in range(wl.n_kv_heads):
        for b in range(wl.batch):
            got, want = idx[g, cu_keep[b]:cu_keep[b + 1]], want_idx[g, cu_keep[b]:cu_keep[b + 1]]
            if np.array_equal(got, want):
                continue
            row = oI[g, wl.cu_seqlens_k[b]:wl.cu_seqlens_k[b + 1]]
            tau = row[want].min()
            for j in np.setxor1d(got, want):
                if 0 <= j < len(row) and abs(row[j] - tau) <= REL * abs(tau):
                    tie_swaps += 1
                else:
                    beyond_ties += 1
    mask_ok = bool(np.array_equal(mask.sum(axis=1), np.full(wl.n_kv_heads, int(wl.k_keep.sum()))))
    finite = bool(np.isfinite(O).all() and np.isfinite(lse).all() and np.isfinite(imp).all())
    ok = finite and o_err <= O_ATOL and l_rel <= REL and i_rel <= REL and beyond_ties == 0 and mask_ok
    return {"ok": bool(ok), "rows_checked": int(len(rows)), "o_max_abs": round(o_err, 5),
            "lse_rel": float(f"{l_rel:.3g}"), "importance_rel": float(f"{i_rel:.3g}"),
            "index_diffs_beyond_ties": beyond_ties, "index_swaps_inside_ties": tie_swaps}


def mfma_probe(iters=40000, reps=3):
    """What the bf16 matrix pipe sustains by itself (libpdd_probe.so), on constant operands and on
    operands that change from one MFMA to the next: TFLOP/s and the clock this implies."""
    import numpy as np
    import torch
    path = os.path.join(ROOT, "paper_2508_09035_amd", "libpdd_probe.so")
    if not os.path.exists(path):
        raise RuntimeError(f"{path} is not built; run __graft_entry__.build()")
    lib = ctypes.CDLL(path)
    lib.pdd_probe_operand_bytes.restype = ctypes.c_int
    lib.pdd_probe_mfma_flops.restype = ctypes.c_double
    lib.pdd_probe_mfma_flops.argtypes = [ctypes.c_int, ctypes.c_int]
    lib.pdd_probe_mfma.restype = ctypes.c_int
    lib.pdd_probe_mfma.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p,
                                   ctypes.c_void_p, ctypes.c_void_p]
    blocks = torch.cuda.get_device_properties(0).multi_processor_count
    nbytes = lib.pdd_probe_operand_bytes()
    rng = np.random.default_rng(7)
    import workloads
    bits = workloads.f32_to_bf16_bits(rng.standard_normal(nbytes // 2).astype(np.float32))
    operands = torch.from_numpy(bits.view(np.int16)).cuda()
    sink = torch.empty(blocks * 512, dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream or None
    out = {}
    for name, varying in (("constant_operands", 0), ("varying_operands", 1)):
        def launch():
            rc = lib.pdd_probe_mfma(varying, blocks, iters, operands.data_ptr(), sink.data_ptr(), stream)
            if rc != 0:
                raise RuntimeError(f"probe launch failed: hipError {rc}")
        ms = time_gpu(launch, reps, 1)
        # a SIMD's matrix pipe needs 32 cycles per MFMA and serves two waves of 8 MFMAs per iteration
        # here, so the run cannot have been clocked lower than this (the counters under profiles/
        # show the pipe 95-99 % busy, i.e. the bound is nearly tight)
        pipe_cycles = iters * 8 * 2 * 32
        out[name] = {"tflops": round(lib.pdd_probe_mfma_flops(blocks, iters) / (ms * 1e-3) / 1e12, 1),
                     "min_clock_ghz": round(pipe_cycles / (ms * 1e-3) / 1e9, 3)}
    return out


def select_scaled(spec, steps):
    """The selection kernel alone at streaming size: `rows x n` seeded fp32 scores (rows as
    sequences of one head row, keep 1/10), algorithmic bytes = 4 B per score + 4 B per kept index +
    1 B per mask byte."""
    import numpy as np
    import torch
    import paper_2508_09035_amd as pdd
    rows, n = (int(x) for x in spec.lower().split("x"))
    g = torch.Generator(device="cuda").manual_seed(5)
    scores = torch.rand((1, rows * n), generator=g, device="cuda") ** 6
    keep = max(1, n // 10)
    cu_k = torch.arange(0, rows + 1, dtype=torch.int32, device="cuda") * n
    k_per = torch.full((rows,), keep, dtype=torch.int32, device="cuda")
    cu_keep = torch.arange(0, rows + 1, dtype=torch.int32, device="cuda") * keep
    idx = torch.empty((1, rows * keep), dtype=torch.int32, device="cuda")
    mask = torch.empty((1, rows * n), dtype=torch.uint8, device="cuda")
    ms = time_gpu(lambda: pdd.select_topk(scores, cu_k, n, k_per, cu_keep, rows * keep, idx, mask), steps, 2)
    nbytes = rows * (4 * n + 4 * keep + n)
    assert int(mask.sum().item()) == rows * keep
    return {"select_scaled": spec, "ms": round(ms, 4), "algorithmic_bytes": nbytes,
            "GBps": round(nbytes / (ms * 1e-3) / 1e9, 1), "frac_of_hbm_peak": round(nbytes / (ms * 1e-3) / 1e9 / PEAK_HBM_GBS, 4)}


def run_config(name, args, budget_gflop, with_cpu_baseline):
    import torch
    import workloads
    import paper_2508_09035_amd as pdd
    from paper_2508_09035_amd.harness import DeviceWorkload

    wl = workloads.make_workload(name)
    dev = DeviceWorkload(wl)
    pdd.set_option(pdd.OPT_ATTN_WAVES, args.waves)

    res = {}
    if not args.no_parity:
        rows, oO, oL, flops, dt = oracle_sample(wl, budget_gflop)
        res["parity"] = parity(wl, dev, rows, oO, oL)
        if with_cpu_baseline:
            import oracle
            res["cpu_baseline"] = {
                "value": flops / dt / 1e12, "unit": "TFLOP/s", "cores": oracle.num_threads(), "kind": "oracle",
                "sample": f"{len(rows)} seeded random query rows x {wl.n_q_heads} heads of {wl.name} "
                          f"({flops / 1e9:.1f} GFLOP of attention, fp64, {dt:.1f} s)"}

    # whole path, then per-kernel legs (same launch configuration), HIP events on the launch stream
    ms_step = time_gpu(dev.step, args.steps, args.warmup)
    ms_attn = time_gpu(lambda: dev.attn(with_importance=False), args.steps, 2)
    ms_attn_median, ms_attn_min = time_gpu_each(lambda: dev.attn(with_importance=False), args.steps)
    ms_attn_imp = time_gpu(lambda: dev.attn(with_importance=True), args.steps, 2)
    ms_select = time_gpu(dev.select, args.steps, 2)

    attn_flops, imp_flops = wl.attn_flops(), wl.importance_flops()
    tflops_path = (attn_flops + imp_flops) / (ms_step * 1e-3) / 1e12
    tflops_attn = attn_flops / (ms_attn * 1e-3) / 1e12
    sel_bytes = 4 * wl.n_kv_heads * int((wl.cand_end - wl.cand_begin).sum()) \
        + 4 * wl.n_kv_heads * int(wl.k_keep.sum()) + wl.n_kv_heads * wl.total_k
    t = TRAFFIC.get(wl.name)
    traffic = t["bytes"] if t and t["sources_sha256"] == kernel_digest() else None
    res.update({
        "value": round(tflops_path, 2),
        "ms_per_step": round(ms_step, 4),
        "config": {"workload": f"{wl.name}: {wl.notes}", "batch": wl.batch,
                   "total_q": wl.total_q, "total_k": wl.total_k, "n_q_heads": wl.n_q_heads,
                   "n_kv_heads": wl.n_kv_heads, "head_dim": wl.head_dim, "window": wl.window,
                   "keep_ratio": str(wl.keep_ratio), "parallelism": "single GPU"},
        "pct_bf16_mfma_peak": round(100 * tflops_path / PEAK_BF16_TFLOPS, 2),
        "prompt_tokens_per_s": round(wl.total_q / (ms_step * 1e-3), 1),
        "legs_ms": {"attention": round(ms_attn, 4), "attention+importance": round(ms_attn_imp, 4),
                    "select+compaction": round(ms_select, 4)},
        "select_GBps": round(sel_bytes / (ms_select * 1e-3) / 1e9, 2),
        "roofline": {"bound": "mfma",
                     "kernel": {pdd.ATTN_WIDE: "attn_wide_kernel", pdd.ATTN_ROWS: "attn_rows_kernel"}.get(dev.attn_form(False), "attn_fwd_kernel"),
                     "achieved": round(tflops_attn, 2), "peak": PEAK_BF16_TFLOPS,
                     "unit": "TFLOP/s", "frac": round(tflops_attn / PEAK_BF16_TFLOPS, 4),
                     "traffic": traffic,
                     # single launches of the same kernel, one event pair each (frac is the mean above)
                     "ms_median": round(ms_attn_median, 4), "ms_min": round(ms_attn_min, 4),
                     "frac_at_min": round(attn_flops / (ms_attn_min * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 4)},
    })
    del dev
    torch.cuda.empty_cache()
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--config", default="all",
                    help="all (default): the 32k-token prompt as the headline plus the other four "
                         "configurations under `configs`; or one of c1..c5 alone")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-parity", action="store_true", help="skip the in-run comparison with the oracle")
    ap.add_argument("--no-probe", action="store_true", help="skip the matrix-pipe probe")
    ap.add_argument("--probe-only", action="store_true", help="run only the matrix-pipe probe")
    ap.add_argument("--select-scaled", default="", metavar="ROWSxN",
                    help="run only the selection kernel on ROWS rows of N seeded scores (streaming size)")
    ap.add_argument("--waves", type=int, default=0, help="attention waves per workgroup (0 = auto)")
    ap.add_argument("--kernel-digest", action="store_true", help="print the digest of the attention "
                    "kernel sources (the key of the stored HBM traffic figure) and exit")
    ap.add_argument("--calibration-copy-mib", type=int, default=0,
                    help="after the timed legs also run one plain device copy of this many MiB "
                         "(a known-size reference for HBM byte counters)")
    args = ap.parse_args()
    if args.kernel_digest:
        print(kernel_digest())
        return
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (no sharding, no collectives); "
              "use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2508_09035_amd as pdd

    pdd.load_library()                      # fails loudly if the HIP library is not built
    torch.cuda.set_device(0)

    if args.probe_only:
        print(json.dumps({"measured_peak": mfma_probe()}))
        return
    if args.select_scaled:
        print(json.dumps(select_scaled(args.select_scaled, args.steps)))
        return

    headline = HEADLINE if args.config == "all" else args.config
    with_cpu = not args.no_cpu_baseline and not args.no_parity
    head = run_config(headline, args, 200.0, with_cpu)
    others = {}
    if args.config == "all":
        for name in OTHERS:
            r = run_config(name, args, 15.0, False)
            others[name] = {k: r[k] for k in ("value", "ms_per_step", "pct_bf16_mfma_peak",
                                              "prompt_tokens_per_s", "legs_ms", "roofline", "parity")
                            if k in r}

    if args.calibration_copy_mib > 0:
        src = torch.ones(args.calibration_copy_mib << 20, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    out = {
        "metric": "causal prefill attn TFLOP/s (+importance) & % bf16 MFMA peak; prompt tokens/s",
        "value": head["value"], "unit": "TFLOP/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
    }
    for k in ("config", "pct_bf16_mfma_peak", "prompt_tokens_per_s", "legs_ms", "select_GBps", "roofline"):
        out[k] = head[k]
    if not args.no_probe:
        out["roofline"]["measured_peak"] = mfma_probe()
    if "cpu_baseline" in head:
        out["cpu_baseline"] = head["cpu_baseline"]
    ok = True
    if not args.no_parity:
        out["parity"] = head["parity"]
        ok = head["parity"]["ok"] and all(o["parity"]["ok"] for o in others.values())
        out["parity_ok"] = bool(ok)
    if others:
        out["configs"] = others
    print(json.dumps(out))
    if not ok:
        print("bench.py: the in-run comparison with the oracle FAILED (see `parity`)", file=sys.stderr)
        sys.exit(1)


if __name__ == "__main__":
    main()

# Field notes
#   value / unit   whole-path throughput: (attention + importance flops, causal-halved,
#                  4*d per visible pair + 2*d per window pair) / step time
#   roofline       the attention kernel alone: algorithmic flops per launch / its
#                  average duration between HIP events, against the dense bf16 MFMA peak
#                  traffic = HBM bytes per launch from byte counters (null when not measured for
#                  these kernel sources)
#                  measured_peak = the matrix pipe alone (probe kernel), constant and varying operands,
#                  with the lowest clock the run can have had (pipe cycles needed / duration)
#   parity         outputs of one step against the CPU oracle on the same tensors, before timing
#   configs        the same measurements for the other configurations (not the headline)
#   cpu_baseline   the fp64 oracle timed on a bounded sample of rows (reported, not a target)
