#!/usr/bin/env python3
"""Throughput of ring-chunked attention (forward + recompute backward) on one MI355X.

One step = one pass of the whole hot path over one batch of resident synthetic input:
ringx_attn_fwd (every K/V chunk streamed, per-chunk local results merged by Eq. (5) in registers)
followed by ringx_attn_bwd (preprocess D = rowsum(dO * O), then the recompute backward with dQ
accumulated over every chunk).  The default workload is one GPU's share of an 8-way ring:
B=1, H=16, d=128, a query shard of 32,768 tokens against all 262,144 keys (a 64^3 token grid) in
R=8 chunks, bf16 storage, Q/K/V/dO ~ N(0,1)/sqrt(2).

Throughput counts 12*B*H*Nq*Nk*d flops per step (4 in the forward's two contractions, 8 in the
backward's four; the backward's recomputation of the scores is not credited).  Prints one JSON
line on stdout; progress goes to stderr.

    python bench.py [--gpus 1] [--steps 10] [--warmup 2] [--no-cpu-baseline]
"""

from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "attention fwd+bwd TFLOP/s and % of bf16 MFMA peak at Nk=262,144, 1 GPU"
PEAK_BF16_TFLOPS = 2516.6     # 256 CUs x 2.4 GHz x 4096 dense bf16 flop/clk/CU
PEAK_HBM_GBS = 8000.0


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def _code_only(text):
    """C++ source without its comments and blank space, so that a change of wording does not
    retire the counters taken on the same code (string literals here hold no comment markers)."""
    import re
    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    return " ".join(text.split())


def kernel_source_hash(files):
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(ROOT, "paper_2507_16697_amd", "csrc", f)) as fh:
            h.update(_code_only(fh.read()).encode())
    return h.hexdigest()[:16]


def load_traffic(kernel, workload, src_hash):
    """Measured HBM traffic of a kernel (rocprofv3 FETCH_SIZE / WRITE_SIZE), if it was taken on
    the kernel's current source; otherwise None."""
    path = os.path.join(ROOT, "profiles", f"traffic_{kernel}_{workload}.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        rec = json.load(f)
    if rec.get("source_hash") != src_hash:
        return None
    return rec.get("bytes_per_launch")


def _dkdv_dispatches(bhkv, Nk, R):
    """Kernel launches per ringx_attn_bwd_dkdv call at d = 128 (the library's grouping of K/V
    heads: about 4096 workgroups of 128 keys per launch)."""
    tpc = -(-(-(-Nk // R)) // 128)
    per = max(1, 4096 // (R * tpc))
    return -(-bhkv // per)


def _oracle_fwd_bwd(inputs, oracle, t, w, h, rows, with_bwd=True):
    """Seconds of the fp64 oracle, as it stands, on head h: queries 0..rows-1 against all keys,
    forward (+ backward).  Returns (seconds, flops of the 4 (+8) * rows * Nk * d convention)."""
    import numpy as np

    store = w.dtype
    q = inputs.to_f64(t["q"][0, h, :rows], store)
    k = inputs.to_f64(t["k"][0, h], store)
    v = inputs.to_f64(t["v"][0, h], store)
    t0 = time.perf_counter()
    o, lse = oracle.head_attention(q, k, v, w.scale)
    flops = 4.0 * rows * w.Nk * w.d
    if with_bwd:
        do = inputs.to_f64(t["do"][0, h, :rows], store)
        D = oracle.head_bwd_preprocess(o, do)
        dq, dk, _ = oracle.head_attention_bwd(q, k, v, do, lse, D, w.scale)
        assert np.all(np.isfinite(dq)) and np.all(np.isfinite(dk))
        flops = 12.0 * rows * w.Nk * w.d
    return time.perf_counter() - t0, flops


def cpu_baseline(t, w, rows, full_head=False, others=True):
    """The fp64 oracle on the host cores this process may use (len(os.sched_getaffinity(0)), the
    BLAS library held to that many threads; numpy's elementwise work is single-threaded).

    The headline sample: head 0 of the timed workload, its first `rows` queries against all keys,
    forward + backward; the whole step's oracle time is that times (Nq / rows) * B * H (every row
    of every head costs the same), reported as an extrapolation.  Beside it: the tiny exactness
    case in full (forward, on all cores and on one core) and one full head of the 16k single shard
    (forward + backward, extrapolated to its 16 heads).  full_head=True also times one full head
    of the timed workload and the whole single shard (minutes)."""
    from threadpoolctl import threadpool_info, threadpool_limits

    import oracle
    from paper_2507_16697_amd import inputs

    cores = len(os.sched_getaffinity(0))
    rec = {"unit": "TFLOP/s", "kind": "oracle", "cores": cores, "cpu": _cpu_model()}
    with threadpool_limits(limits=cores, user_api="blas"):
        blas = max([p.get("num_threads", 1) for p in threadpool_info()
                    if p.get("user_api") == "blas"] or [1])
        sec, flops = _oracle_fwd_bwd(inputs, oracle, t, w, 0, rows)
        steps = w.B * w.H * (w.Nq / rows)
        rec.update({
            "value": flops / sec / 1e12, "seconds": sec, "blas_threads": blas,
            "sample": f"fp64 oracle, head 0 of {w.name}: queries 0..{rows - 1} against all "
                      f"{w.Nk} keys, forward + backward, {flops:.3e} flops (12*rows*Nk*d)",
            "step_seconds_extrapolated": sec * steps,
            "extrapolation": f"x {steps:g} = (Nq / rows) * B * H: every row of every head costs "
                             "the same",
        })
        extra = {}
        if not others:
            return rec
        w1 = inputs.WORKLOADS["exact_fp32_n1k"]
        t1 = inputs.make_workload(w1.name)
        s_all = sum(_oracle_fwd_bwd(inputs, oracle, t1, w1, h, w1.Nq, with_bwd=False)[0]
                    for h in range(w1.H))
        with threadpool_limits(limits=1, user_api="blas"):
            s_one = sum(_oracle_fwd_bwd(inputs, oracle, t1, w1, h, w1.Nq, with_bwd=False)[0]
                        for h in range(w1.H))
        f1 = 4.0 * w1.B * w1.H * w1.Nq * w1.Nk * w1.d
        extra[w1.name] = {"pass": "fwd", "seconds": s_all, "tflops": f1 / s_all / 1e12,
                          "seconds_1_core": s_one, "tflops_1_core": f1 / s_one / 1e12,
                          "what": "in full (every head, every row)"}
        w2 = inputs.WORKLOADS["shard_n16k_d64"]
        t2 = inputs.make_workload(w2.name)
        s2, f2 = _oracle_fwd_bwd(inputs, oracle, t2, w2, 0, w2.Nq)
        extra[w2.name] = {"pass": "fwd+bwd", "seconds_head0": s2, "tflops": f2 / s2 / 1e12,
                          "seconds_extrapolated": s2 * w2.B * w2.H,
                          "what": f"head 0 in full, x {w2.B * w2.H} heads extrapolated"}
        if full_head:
            sf, ff = _oracle_fwd_bwd(inputs, oracle, t, w, 0, w.Nq)
            extra[w.name + "_head0_full"] = {
                "pass": "fwd+bwd", "seconds": sf, "tflops": ff / sf / 1e12,
                "step_seconds_extrapolated": sf * w.B * w.H,
                "what": f"head 0 in full, x {w.B * w.H} heads extrapolated"}
            sa = s2 + sum(_oracle_fwd_bwd(inputs, oracle, t2, w2, h, w2.Nq)[0]
                          for h in range(1, w2.H))
            extra[w2.name]["seconds_full"] = sa
        rec["other_configs"] = extra
    return rec


def input_sha256(t):
    """SHA-256 of every generated input tensor (host storage bytes), computed in parallel."""
    import concurrent.futures

    from paper_2507_16697_amd import inputs

    names = sorted(t)
    with concurrent.futures.ThreadPoolExecutor(len(names)) as ex:
        digests = list(ex.map(lambda n: inputs.sha256_of(t[n]), names))
    return dict(zip(names, digests))


class ClockSampler:
    """Samples the GPU's shader clock (rocm-smi) on a host thread while the timed steps run."""

    def __init__(self, period=0.5, enabled=True):
        import threading
        self.enabled = enabled
        self.period = period
        self.samples = []
        self.error = None
        self._stop = threading.Event()
        self._thread = threading.Thread(target=self._run, daemon=True)

    def _read(self):
        import re
        import subprocess
        r = subprocess.run(["rocm-smi", "--showclocks", "--json"], capture_output=True,
                           text=True, timeout=10)
        data = json.loads(r.stdout)
        for card in data.values():
            for key, val in card.items():
                if "sclk" in key.lower():
                    m = re.search(r"(\d+)\s*Mhz", str(val), re.I)
                    if m:
                        return int(m.group(1))
        raise ValueError("no sclk in rocm-smi output")

    def _run(self):
        while not self._stop.is_set():
            try:
                self.samples.append(self._read())
            except Exception as e:   # a missing or failing tool leaves the record empty
                self.error = f"{type(e).__name__}: {e}"[:200]
                return
            self._stop.wait(self.period)

    def __enter__(self):
        if self.enabled:
            self._thread.start()
        else:
            self.error = "not sampled (--no-sclk)"
        return self

    def __exit__(self, *exc):
        self._stop.set()
        if self.enabled:
            self._thread.join(timeout=15)

    def record(self):
        if not self.samples:
            return {"source": "rocm-smi --showclocks", "mhz": None, "error": self.error}
        x = sorted(self.samples)
        return {"source": "rocm-smi --showclocks, sampled every 0.5 s over the timed steps",
                "samples": len(x), "mhz_min": x[0], "mhz_median": x[len(x) // 2],
                "mhz_max": x[-1]}


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _time(torch, stream, fn, warmup, n):
    """Per-call milliseconds of fn (HIP events on `stream`): sorted list of n values."""
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(n)]
    for a, b in ev:
        a.record(stream)
        fn()
        b.record(stream)
    torch.cuda.synchronize()
    return sorted(a.elapsed_time(b) for a, b in ev)


def _stats(ms, flops):
    med = ms[len(ms) // 2]
    return {"ms_min": ms[0], "ms_median": med, "ms_max": ms[-1], "calls": len(ms),
            "tflops_median": flops / (med * 1e-3) / 1e12,
            "frac_median": flops / (med * 1e-3) / 1e12 / PEAK_BF16_TFLOPS}


def other_shapes(torch, np, inputs, ringx, stream, dev):
    """Timings of the other paper-shaped workloads: the 16k single shard (fwd+bwd, d=64) and the
    turbulence tokens (fwd, d=64: 256^3 field, 4^3 patches, seeded embedding and projections),
    both from the host recipe, and the 524k long step (fwd+bwd, d=128, plus the standalone
    merge), whose 2.4e9 inputs are drawn on the device (torch's seeded generator, the workload's
    distribution; labelled so in the record) so that the run stays short; its parity tests use
    the host recipe."""
    res = {}
    gen = torch.Generator(device=dev)

    def iid(w, seed):
        gen.manual_seed(seed)
        bf = dict(dtype=torch.bfloat16, device=dev)
        x = {n: (torch.randn((w.B, w.H, N, w.d), generator=gen, device=dev) * w.std).to(**bf)
             for n, N in (("q", w.Nq), ("k", w.Nk), ("v", w.Nk))}
        x["do"] = (torch.randn((w.B, w.H, w.Nq, w.d), generator=gen, device=dev)
                   * w.do_std).to(**bf)
        return x

    def fwd_bwd(w, x, warmup, n):
        q, k, v, do = x["q"], x["k"], x["v"], x["do"]
        B, H, Nq, Nk, d, R = w.B, w.H, w.Nq, w.Nk, w.d, w.R
        out = torch.empty_like(q)
        lse = torch.empty((B, H, Nq), dtype=torch.float32, device=dev)
        delta = torch.empty((2, B, H, Nq), dtype=torch.float32, device=dev)
        dq = torch.empty((B, H, Nq, d), dtype=torch.float32, device=dev)
        dk = torch.empty((B, H, Nk, d), dtype=torch.float32, device=dev)
        dv = torch.empty_like(dk)

        def step():
            ringx.ringx_attn_fwd(q, k, v, R, scale=w.scale, out=out, lse=lse, stream=stream)
            ringx.ringx_bwd_preprocess(out, do, lse, delta=delta, stream=stream)
            ringx.ringx_attn_bwd_dkdv(q, k, v, do, lse, delta, R, scale=w.scale, dk=dk, dv=dv,
                                      stream=stream)
            ringx.ringx_attn_bwd_dq(q, k, v, do, lse, delta, R, scale=w.scale, dq=dq,
                                    stream=stream)

        r = _stats(_time(torch, stream, step, warmup, n), 6 * w.gemm_unit())
        r.update(workload=w.name, B=B, H=H, Nq=Nq, Nk=Nk, d=d, R=R, passes="fwd+bwd",
                 flops=6 * w.gemm_unit(), inputs="device-drawn i.i.d., the workload's distribution")
        if not bool(torch.isfinite(dq).all()):
            raise RuntimeError(f"non-finite results at {w.name}")
        return r

    w = inputs.WORKLOADS["shard_n16k_d64"]
    tt = inputs.make_workload(w.name)
    x = {n: torch.from_numpy(np.ascontiguousarray(tt[n]).view(np.int16)).to(dev)
         .view(torch.bfloat16) for n in ("q", "k", "v", "do")}
    del tt
    res[w.name] = fwd_bwd(w, x, 3, 10)
    res[w.name]["inputs"] = "host recipe"
    del x
    log(f"[bench] {w.name}: {res[w.name]['ms_median']:.2f} ms/step, "
        f"{res[w.name]['tflops_median']:.1f} TFLOP/s")

    w = inputs.WORKLOADS["turbulence_nk262k_d64"]
    t0 = time.time()
    tt = inputs.make_workload(w.name)
    log(f"[bench] {w.name} inputs (host recipe) in {time.time() - t0:.1f}s")
    q, k, v = (torch.from_numpy(np.ascontiguousarray(tt[n]).view(np.int16)).to(dev)
               .view(torch.bfloat16) for n in ("q", "k", "v"))
    del tt
    out = torch.empty_like(q)
    lse = torch.empty((w.B, w.H, w.Nq), dtype=torch.float32, device=dev)
    ms = _time(torch, stream, lambda: ringx.ringx_attn_fwd(q, k, v, w.R, scale=w.scale, out=out,
                                                           lse=lse, stream=stream), 1, 5)
    res[w.name] = _stats(ms, 2 * w.gemm_unit())
    res[w.name].update(workload=w.name, B=w.B, H=w.H, Nq=w.Nq, Nk=w.Nk, d=w.d, R=w.R,
                       passes="fwd", flops=2 * w.gemm_unit(), inputs="host recipe")
    log(f"[bench] {w.name}: {res[w.name]['ms_median']:.2f} ms/fwd, "
        f"{res[w.name]['tflops_median']:.1f} TFLOP/s")
    del q, k, v, out, lse

    w = inputs.WORKLOADS["long_nk524k_d128"]
    x = iid(w, w.seed)
    res[w.name] = fwd_bwd(w, x, 1, 5)
    log(f"[bench] {w.name}: {res[w.name]['ms_median']:.1f} ms/step, "
        f"{res[w.name]['tflops_median']:.1f} TFLOP/s")
    po, pl = ringx.ringx_attn_fwd_partials(x["q"], x["k"], x["v"], w.R, scale=w.scale,
                                           stream=stream)
    mo = torch.empty_like(x["q"])
    ml = torch.empty((w.B, w.H, w.Nq), dtype=torch.float32, device=dev)
    ms = _time(torch, stream, lambda: ringx.ringx_lse_merge(po, pl, out=mo, lse=ml, stream=stream),
               2, 10)
    rows = w.B * w.H * w.Nq
    mbytes = w.R * rows * (4 * w.d + 4) + rows * (2 * w.d + 4)
    med = ms[len(ms) // 2]
    res[w.name]["lse_merge"] = {"ms_median": med, "bytes": mbytes,
                                "GB/s": mbytes / (med * 1e-3) / 1e9,
                                "frac": mbytes / (med * 1e-3) / 1e9 / PEAK_HBM_GBS}
    log(f"[bench] {w.name} lse_merge {med:.3f} ms, {mbytes / (med * 1e-3) / 1e9:.0f} GB/s")
    del x, po, pl, mo, ml
    return res


# ------------------------------------------------------------------------------------------------
# rocprofv3 outputs -> profiles/ summaries (CPU only; the commands that make the outputs are written
# into each summary)

PROFILE_STEP = ("python -u bench.py --steps 1 --warmup 0 --no-cpu-baseline --no-ring --no-gqa --no-stored-ds "
                "--no-tokenizer --no-shapes --no-sclk")
PROFILE_TRACE = ("python -u bench.py --steps 3 --warmup 1 --no-cpu-baseline --no-ring --no-gqa --no-stored-ds "
                 "--no-tokenizer --no-shapes --no-sclk")
# the step with the backward through stored dS (run once after one plain step)
PROFILE_DS = ("python -u bench.py --steps 1 --warmup 0 --no-cpu-baseline --no-ring --no-gqa "
              "--no-merge --no-tokenizer --no-shapes --no-sclk")
BUSY_COUNTERS = ("SQ_VALU_MFMA_BUSY_CYCLES SQ_VALU_MFMA_COEXEC_CYCLES SQ_BUSY_CYCLES "
                 "SQ_LDS_IDX_ACTIVE SQ_LDS_BANK_CONFLICT SQ_INSTS_LDS GRBM_GUI_ACTIVE")
# L2 (TCC) hits and misses of the step's kernels (one counter pass; two of the four TCC counters)
L2_COUNTERS = "TCC_HIT_sum TCC_MISS_sum"
# instruction mix and wave states of every matrix kernel of the step and the other shapes (two
# counter passes: at most 8 SQ counters per run)
PROFILE_MIX = ("python -u bench.py --steps 1 --warmup 0 --no-cpu-baseline --no-ring --no-gqa "
               "--no-stored-ds --no-tokenizer --no-sclk --no-merge")
MIX_COUNTERS = [("pmc_stall1", "SQ_WAVE_CYCLES SQ_WAIT_ANY SQ_WAIT_INST_ANY SQ_WAIT_INST_LDS "
                 "SQ_ACTIVE_INST_VALU SQ_ACTIVE_INST_LDS SQ_ACTIVE_INST_ANY SQ_ACTIVE_INST_MISC "
                 "GRBM_GUI_ACTIVE"),
                ("pmc_stall2", "SQ_INSTS_VALU SQ_INSTS_MFMA SQ_INSTS_LDS SQ_INSTS_SALU "
                 "SQ_INSTS_VALU_TRANS_F32 SQ_BUSY_CYCLES SQ_VALU_MFMA_BUSY_CYCLES SQ_INSTS_VMEM "
                 "GRBM_GUI_ACTIVE")]
# matrix kernels of the instruction-mix summary: kernel, template arguments -> label, waves per SIMD
MIX_KERNELS = [("fwd_bf16_kernel", (128, 0, 1, 8), "fwd_bf16_kernel<128, fused merge>", 2),
               ("bwd_dkdv_kernel", (128, False), "bwd_dkdv_kernel<128>", 1),
               ("bwd_dq_kernel", (128,), "bwd_dq_kernel<128>", 1),
               ("fwd_bf16_kernel", (64, 0, 1, 8), "fwd_bf16_kernel<64, fused merge>", 2),
               ("fwd_bf16_kernel", (64, 0, 1, 4), "fwd_bf16_kernel<64, fused merge>, half-size", 3),
               ("bwd_dkdv_kernel", (64, 8, 1), "bwd_dkdv_kernel<64>", 4),
               ("bwd_dq_kernel", (64, 1, 8, 64), "bwd_dq_kernel<64>", 2),
               ("bwd_dq_kernel", (64, 1, 4, 32), "bwd_dq_kernel<64>, half-size", 3)]

# kernel, template arguments -> (label in the summaries, traffic key, source files of its hash): the
# forms that the full launches of the profiled workload take
PROFILE_KERNELS = [
    ("fwd_bf16_kernel", (128, 0, 1, 8), "fwd_bf16_kernel<128, fused merge>", "fwd_bf16",
     ["fwd_bf16.hip", "ringx_device.h"]),
    ("fwd_bf16_kernel", (128, 1, 1, 8), "fwd_bf16_kernel<128, partials>", "fwd_bf16_partials",
     ["fwd_bf16.hip", "ringx_device.h"]),
    ("bwd_dkdv_kernel", (128, False), "bwd_dkdv_kernel<128>", "bwd_dkdv",
     ["bwd_bf16.hip", "ringx_device.h"]),
    ("bwd_dkdv_kernel", (128, True), "bwd_dkdv_kernel<128, dS stores>", "bwd_dkdv_store",
     ["bwd_bf16.hip", "ringx_device.h"]),
    ("bwd_dq_ds_kernel", (), "bwd_dq_ds_kernel", "bwd_dq_ds", ["bwd_dq_ds.hip", "ringx_device.h"]),
    ("bwd_dq_kernel", (128,), "bwd_dq_kernel<128>", "bwd_dq", ["bwd_dq_bf16.hip", "ringx_device.h"]),
    ("bwd_pre_bf16_kernel", (128,), "bwd_pre_bf16_kernel<128>", "bwd_pre",
     ["bwd_pre.hip", "ringx_device.h"]),
    ("merge_vec4_kernel", (True, 1), "merge_vec4_kernel<bf16 out>", "lse_merge",
     ["merge.hip", "ringx_device.h"]),
]


def _is_kernel(name, kernel, args):
    """Whether a traced kernel name, mangled or demangled as rocprofv3 prints it, is this kernel with
    exactly these template arguments."""
    if not args:
        return kernel in name
    mangled = "".join(f"L{'b' if isinstance(a, bool) else 'i'}{int(a)}E" for a in args)
    plain = ", ".join(str(a).lower() for a in args)
    return f"{kernel}I{mangled}E" in name or f"{kernel}<{plain}>" in name


def _profile_kernel(name):
    for kernel, args, label, key, files in PROFILE_KERNELS:
        if _is_kernel(name, kernel, args):
            return label, key, files
    return None


def _read_csv(path):
    import csv
    with open(path, newline="") as f:
        return list(csv.DictReader(f))


def _pmc_per_dispatch(dirpath, counter):
    """{dispatch id: (kernel name, value)} of one counter from a rocprofv3 --pmc CSV."""
    rows = _read_csv(os.path.join(dirpath, "pmc_counter_collection.csv"))
    out = {}
    for r in rows:
        if r["Counter_Name"] != counter:
            continue
        did = int(r["Dispatch_Id"])
        name, val = out.get(did, (r["Kernel_Name"], 0.0))
        out[did] = (name, val + float(r["Counter_Value"]))
    return out


def summarize_profiles(root, workload):
    from paper_2507_16697_amd import inputs
    w = inputs.WORKLOADS[workload]
    B, H, Nq, Nk, d, R = w.B, w.H, w.Nq, w.Nk, w.d, w.R
    rows = B * H * Nq
    shape = f"B={B}, H={H}, Nq={Nq}, Nk={Nk}, d={d}, R={R}, bf16"
    prof = os.path.join(ROOT, "profiles")
    cmd = lambda d_, o, extra: f"rocprofv3 {extra} --output-format csv -d gpurun_out/{d_} -o {o} -- "

    # kernel trace
    stats = _read_csv(os.path.join(root, "prof_trace", "ring8_kernel_stats.csv"))
    lines = []
    for r in stats:
        k = _profile_kernel(r["Name"])
        if k:
            lines.append((k[0], int(r["Calls"]), float(r["AverageNs"]), float(r["MinNs"]),
                          float(r["MaxNs"])))
    lines.sort(key=lambda x: -x[2])
    # dispatches per call of each entry point (dK/dV is launched two K/V heads at a time): the
    # trace's calls over the fused forward's, one of which runs per step
    calls_of = {lab: c for lab, c, _, _, _ in lines}
    per_step = calls_of.get("fwd_bf16_kernel<128, fused merge>", 1) or 1
    per_call = {lab: max(1, round(c / per_step)) for lab, c, _, _, _ in lines
                if lab.startswith("bwd_dkdv")}
    bench_line = None
    log_path = os.path.join(root, "prof_trace.log")
    if os.path.exists(log_path):
        for line in open(log_path):
            if line.startswith("{") and '"metric"' in line:
                bench_line = json.loads(line)
    md = [f"# Kernel trace: {workload} ({shape})", "",
          "Command (run from the repository root on one MI355X):", "",
          "    " + cmd("prof_trace", "ring8", "--kernel-trace --stats") + PROFILE_TRACE, "",
          "The run makes 4 forward and 4 backward passes (1 warmup + 3 timed; each backward = "
          "preprocess + dK/dV + dQ), 1 partials forward and 11 standalone merges.  Durations in ns; "
          "only libringx kernels are listed.  A call of ringx_attn_bwd_dkdv launches its kernel "
          "once per two K/V heads; the last column is the time per call.", "",
          "| kernel | dispatches | average ns per dispatch | min ns | max ns | dispatches per call "
          "| ms per call |", "|---|---|---|---|---|---|---|"]
    md += [f"| {a} | {c} | {avg:.0f} | {mn:.0f} | {mx:.0f} | {per_call.get(a, 1)} | "
           f"{avg * per_call.get(a, 1) / 1e6:.2f} |" for a, c, avg, mn, mx in lines]
    if bench_line:
        c = bench_line["config"]
        md += ["", f"bench.py in the same run (HIP events around each call, "
               f"{bench_line['steps']} timed steps): step {bench_line['ms_per_step']:.2f} ms = fwd "
               f"{c['fwd_ms']:.2f} + preprocess {c['bwd_pre_ms']:.3f} + dK/dV {c['bwd_dkdv_ms']:.2f} "
               f"+ dQ {c['bwd_dq_ms']:.2f} ms; {bench_line['value']:.1f} TFLOP/s "
               f"(12*B*H*Nq*Nk*d per step) = {100 * bench_line['value'] / PEAK_BF16_TFLOPS:.2f}% of "
               f"{PEAK_BF16_TFLOPS}."]
    with open(os.path.join(prof, f"kernel_trace_{workload}.md"), "w") as f:
        f.write("\n".join(md) + "\n")

    # HBM traffic: FETCH_SIZE / WRITE_SIZE per dispatch, calibrated on the 1 GiB copy
    fetch = _pmc_per_dispatch(os.path.join(root, "pmc_FETCH_SIZE"), "FETCH_SIZE")
    write = _pmc_per_dispatch(os.path.join(root, "pmc_WRITE_SIZE"), "WRITE_SIZE")
    cf = _pmc_per_dispatch(os.path.join(root, "pmc_copy_FETCH_SIZE"), "FETCH_SIZE")
    cw = _pmc_per_dispatch(os.path.join(root, "pmc_copy_WRITE_SIZE"), "WRITE_SIZE")
    copy_bytes = 1 << 30
    cf_kib = sorted(v for _, v in cf.values())[len(cf) // 2]
    cw_kib = sorted(v for _, v in cw.values())[len(cw) // 2]
    ff, wf = copy_bytes / (cf_kib * 1024), copy_bytes / (cw_kib * 1024)
    es = 2
    alg = {
        "fwd_bf16": rows * d * es + 2 * B * H * Nk * d * es + rows * d * es + rows * 4,
        "fwd_bf16_partials": rows * d * es + 2 * B * H * Nk * d * es + R * rows * (4 * d + 4),
        "bwd_dkdv": 2 * B * H * Nk * d * es + 2 * rows * d * es + 2 * rows * 4
        + 2 * B * H * Nk * d * 4,
        "bwd_dq": 2 * B * H * Nk * d * es + 2 * rows * d * es + 2 * rows * 4 + rows * d * 4,
        "bwd_pre": 2 * rows * d * es + rows * 4 + 2 * rows * 4,
        "lse_merge": R * rows * (4 * d + 4) + rows * (d * es + 4),
    }
    per_kernel = {}
    for src, which in ((fetch, 0), (write, 1)):
        for did, (name, val) in src.items():
            k = _profile_kernel(name)
            if k:
                per_kernel.setdefault(k[1], ([], [], k[2]))[which].append(val)
    cmds = [cmd("pmc_FETCH_SIZE", "pmc", "--pmc FETCH_SIZE") + PROFILE_STEP,
            cmd("pmc_WRITE_SIZE", "pmc", "--pmc WRITE_SIZE") + PROFILE_STEP,
            cmd("pmc_copy_FETCH_SIZE", "pmc", "--pmc FETCH_SIZE") + "python -u bench.py --copy-probe",
            cmd("pmc_copy_WRITE_SIZE", "pmc", "--pmc WRITE_SIZE") + "python -u bench.py --copy-probe"]
    label_of = {key: lab for _, _, lab, key, _ in PROFILE_KERNELS}
    md = [f"# HBM traffic per call: {workload} ({shape})", "",
          "Counters: `FETCH_SIZE` and `WRITE_SIZE` (KiB per dispatch, L2-to-fabric traffic, so reads "
          "served by", "the MALL count as fetched), each in a run of its own:", ""]
    md += ["    " + c for c in cmds[:2]]
    md += ["", "Calibration: the same counters on a plain 1 GiB device copy (`bench.py --copy-probe`, "
           "3 copies):", ""] + ["    " + c for c in cmds[2:]]
    md += ["", f"The copy reads 1 GiB and writes 1 GiB; FETCH_SIZE reports {cf_kib:.0f} KiB and "
           f"WRITE_SIZE {cw_kib:.0f} KiB, so fetched bytes = FETCH_SIZE x 1024 x {ff:.4f} and written "
           f"bytes = WRITE_SIZE x 1024 x {wf:.4f}.  Per call: the median dispatch times the "
           "dispatches per call (dK/dV: one per two K/V heads).", "",
           "| kernel | FETCH_SIZE KiB | WRITE_SIZE KiB | fetched GB | written GB | traffic GB | "
           "algorithmic GB | traffic / algorithmic |", "|---|---|---|---|---|---|---|---|"]
    for key in ("fwd_bf16", "fwd_bf16_partials", "bwd_dkdv", "bwd_dq", "bwd_pre", "lse_merge"):
        if key not in per_kernel:
            continue
        fv, wv, files = per_kernel[key]
        npc = per_call.get(label_of.get(key), 1)
        fk = sorted(fv)[len(fv) // 2] * npc
        wk = (sorted(wv)[len(wv) // 2] if wv else 0.0) * npc
        fb, wb = fk * 1024 * ff, wk * 1024 * wf
        md.append(f"| {key} | {fk:.0f} | {wk:.0f} | {fb / 1e9:.3f} | {wb / 1e9:.3f} | "
                  f"{(fb + wb) / 1e9:.3f} | {alg[key] / 1e9:.3f} | {(fb + wb) / alg[key]:.2f} |")
        rec = {"kernel": key, "workload": workload, "source_hash": kernel_source_hash(files),
               "fetch_size_kib": fk, "write_size_kib": wk, "fetch_factor": ff, "write_factor": wf,
               "bytes_fetched": fb, "bytes_written": wb, "bytes_per_launch": fb + wb,
               "algorithmic_bytes": alg[key], "commands": cmds}
        with open(os.path.join(prof, f"traffic_{key}_{workload}.json"), "w") as f:
            json.dump(rec, f, indent=1)
            f.write("\n")
    md += ["", "Algorithmic bytes: every input read once and every output written once (fwd: Q, K, "
           "V, out, lse;", "dK/dV: K, V, Q, dO, nl, D, fp32 dK and dV; dQ: K, V, Q, dO, lse, D, fp32 "
           "dQ; preprocess: out, dout, lse,", "D and nl; merge: R fp32 partials and lse, bf16 out and "
           "lse).  Traffic well above it is re-reading", "of K/V (forward, dQ) or Q/dO (dK/dV) that "
           "missed L2."]
    with open(os.path.join(prof, f"hbm_traffic_{workload}.md"), "w") as f:
        f.write("\n".join(md) + "\n")

    # matrix-core, vector and LDS activity from one counter pass
    busy_rows = _read_csv(os.path.join(root, "pmc_busy", "pmc_counter_collection.csv"))
    disp = {}
    for r in busy_rows:
        did = int(r["Dispatch_Id"])
        e = disp.setdefault(did, {"name": r["Kernel_Name"], "t0": int(r["Start_Timestamp"]),
                                  "t1": int(r["End_Timestamp"])})
        e[r["Counter_Name"]] = e.get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
    md = [f"# Matrix-core and LDS activity: {workload} ({shape})", "",
          "Command (run from the repository root on one MI355X, one counter pass):", "",
          "    " + cmd("pmc_busy", "pmc", "--pmc " + BUSY_COUNTERS) + PROFILE_STEP, "",
          "GRBM_GUI_ACTIVE counts GPU clocks summed over the 8 XCDs, so cycles = GRBM_GUI_ACTIVE / 8 "
          "and the", "average shader clock = cycles / kernel duration.  MFMA busy = "
          "SQ_VALU_MFMA_BUSY_CYCLES / (cycles x 1024", "SIMDs); MFMA co-issue = "
          "SQ_VALU_MFMA_COEXEC_CYCLES / SQ_VALU_MFMA_BUSY_CYCLES (matrix-core cycles during", "which "
          "the vector ALU also issued); LDS busy = SQ_LDS_IDX_ACTIVE / (cycles x 256 CUs).  The bf16 "
          "rate the", "matrix cores deliver is MFMA busy x clock / 2.4 GHz x 2516.6 TFLOP/s.", "",
          "| kernel | duration ms | clock GHz | MFMA busy | MFMA co-issue | delivered TFLOP/s | LDS "
          "busy | LDS bank conflicts | LDS instructions |", "|---|---|---|---|---|---|---|---|---|"]
    # the first call of each kernel: its dispatches' durations and counters summed
    first = {}
    for did in sorted(disp):
        e = disp[did]
        k = _profile_kernel(e["name"])
        if not k:
            continue
        agg = first.setdefault(k[0], {"n": 0, "ms": 0.0})
        if agg["n"] >= per_call.get(k[0], 1):
            continue
        agg["n"] += 1
        agg["ms"] += (e["t1"] - e["t0"]) * 1e-6
        for cname, val in e.items():
            if cname.startswith(("SQ_", "GRBM_")):
                agg[cname] = agg.get(cname, 0.0) + val
    for lab, e in first.items():
        k = (lab,)
        ms = e["ms"]
        cyc = e.get("GRBM_GUI_ACTIVE", 0.0) / 8
        ghz = cyc / (ms * 1e6) if ms > 0 else 0.0
        busy = e.get("SQ_VALU_MFMA_BUSY_CYCLES", 0.0) / (cyc * 1024) if cyc else 0.0
        co = (e.get("SQ_VALU_MFMA_COEXEC_CYCLES", 0.0) / e["SQ_VALU_MFMA_BUSY_CYCLES"]
              if e.get("SQ_VALU_MFMA_BUSY_CYCLES") else 0.0)
        lds = e.get("SQ_LDS_IDX_ACTIVE", 0.0) / (cyc * 256) if cyc else 0.0
        md.append(f"| {k[0]} | {ms:.2f} | {ghz:.2f} | {100 * busy:.1f}% | {100 * co:.1f}% | "
                  f"{busy * ghz / 2.4 * PEAK_BF16_TFLOPS:.0f} | {100 * lds:.1f}% | "
                  f"{e.get('SQ_LDS_BANK_CONFLICT', 0.0):.0f} | {e.get('SQ_INSTS_LDS', 0.0):.3e} |")
    md += ["", "Delivered TFLOP/s counts every executed product (the forward 2U, dK/dV 4U with S "
           "recomputed, dQ 3U", "with S and dP recomputed), so it exceeds the credited rates of "
           "bench.py for the two backward kernels."]
    with open(os.path.join(prof, f"mfma_busy_{workload}.md"), "w") as f:
        f.write("\n".join(md) + "\n")
    _summarize_stored_ds(root, workload, w, shape, prof, cmd, ff, wf)
    _summarize_l2(root, workload, shape, prof, cmd, per_call)
    _summarize_instruction_mix(root, workload, prof, cmd)
    # the bench line of a plain `python bench.py` run beside the profiles, if there is one
    full = os.path.join(root, "bench.json")
    if os.path.exists(full):
        for line in open(full):
            if line.startswith("{") and '"metric"' in line:
                bench_line = json.loads(line)
    if bench_line:
        with open(os.path.join(prof, f"bench_{workload}.json"), "w") as f:
            json.dump(bench_line, f, indent=1)
            f.write("\n")
    print(f"wrote summaries of {root} under profiles/")


def _summarize_l2(root, workload, shape, prof, cmd, per_call):
    """L2 hit rate of the first call of each kernel of the step, from the TCC counter pass (when
    it is there).  TCC requests are counted per cache line, whatever the request size."""
    path = os.path.join(root, "pmc_l2", "pmc_counter_collection.csv")
    if not os.path.exists(path):
        return
    disp = {}
    for r in _read_csv(path):
        e = disp.setdefault(int(r["Dispatch_Id"]), {"name": r["Kernel_Name"]})
        e[r["Counter_Name"]] = e.get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
    first = {}
    for did in sorted(disp):
        e = disp[did]
        k = _profile_kernel(e["name"])
        if not k:
            continue
        agg = first.setdefault(k[0], {"n": 0, "hit": 0.0, "miss": 0.0})
        if agg["n"] >= per_call.get(k[0], 1):
            continue
        agg["n"] += 1
        agg["hit"] += e.get("TCC_HIT_sum", 0.0)
        agg["miss"] += e.get("TCC_MISS_sum", 0.0)
    md = [f"# L2 hit rate: {workload} ({shape})", "",
          "Command (run from the repository root on one MI355X, one counter pass):", "",
          "    " + cmd("pmc_l2", "pmc", "--pmc " + L2_COUNTERS) + PROFILE_STEP, "",
          "TCC_HIT_sum and TCC_MISS_sum: requests to the L2 of the 8 XCDs that hit or missed, summed "
          "over", "the dispatches of one call (dK/dV runs as several dispatches per call).  A miss "
          "goes on to the", "memory-side Infinity Cache or HBM; the HBM bytes are in the traffic "
          "summary.", "",
          "| kernel | dispatches | L2 hits | L2 misses | hit rate |", "|---|---|---|---|---|"]
    for lab, e in first.items():
        tot = e["hit"] + e["miss"]
        rate = e["hit"] / tot if tot else 0.0
        md.append(f"| {lab} | {e['n']} | {e['hit']:.4e} | {e['miss']:.4e} | {100 * rate:.1f}% |")
    with open(os.path.join(prof, f"l2_hit_{workload}.md"), "w") as f:
        f.write("\n".join(md) + "\n")


def _summarize_instruction_mix(root, workload, prof, cmd):
    """Instructions per matrix product and wave states of each matrix kernel, summed over all its
    dispatches in the two MIX_COUNTERS passes (when both are there)."""
    paths = [os.path.join(root, d_, "pmc_counter_collection.csv") for d_, _ in MIX_COUNTERS]
    if not all(os.path.exists(p) for p in paths):
        return
    tot = {}
    for p in paths:
        for r in _read_csv(p):
            name = r["Kernel_Name"]
            for kernel, args, label, wps in MIX_KERNELS:
                if _is_kernel(name, kernel, args):
                    e = tot.setdefault(label, {"wps": wps, "disp": set()})
                    e["disp"].add((p, int(r["Dispatch_Id"])))
                    e[r["Counter_Name"]] = e.get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
                    break
    md = [f"# Instruction mix and wave states of the matrix kernels: {workload} and the other "
          "shapes", "", "Commands (run from the repository root on one MI355X, one counter pass "
          "each; the run also makes the", "16k single shard and turbulence-token passes at d = 64 "
          "and the 524k long step):", ""]
    md += ["    " + cmd(d_, "pmc", "--pmc " + c) + PROFILE_MIX for d_, c in MIX_COUNTERS]
    md += ["", "Per matrix product (v_mfma_f32_32x32x16_bf16, 32 cycles of a SIMD's matrix core): "
           "vector-ALU", "instructions other than the products (SQ_INSTS_VALU - SQ_INSTS_MFMA), of "
           "them transcendental", "(SQ_INSTS_VALU_TRANS_F32: the exponentials), LDS and scalar "
           "instructions (s_waitcnt included).", "Wave states as fractions of SQ_WAVE_CYCLES: "
           "waiting on a counter or barrier (SQ_WAIT_ANY), ready but", "not issued (SQ_WAIT_INST_ANY), "
           "issuing vector-ALU (SQ_ACTIVE_INST_VALU, products included) and LDS", "instructions "
           "(SQ_ACTIVE_INST_LDS).  MFMA busy = SQ_VALU_MFMA_BUSY_CYCLES / (GRBM_GUI_ACTIVE / 8 x "
           "1024).", "",
           "| kernel | waves per SIMD | dispatches | VALU / product | exp / product | LDS / product "
           "| scalar / product | MFMA busy | waiting | not issued | VALU active | LDS active |",
           "|---|---|---|---|---|---|---|---|---|---|---|---|"]
    for kernel, args, label, _ in MIX_KERNELS:
        e = tot.get(label)
        if not e or not e.get("SQ_INSTS_MFMA") or not e.get("SQ_WAVE_CYCLES"):
            continue
        m, wc = e["SQ_INSTS_MFMA"], e["SQ_WAVE_CYCLES"]
        # GRBM_GUI_ACTIVE is in both passes: the matrix-core busy fraction uses the second's
        cyc = sum(float(r["Counter_Value"]) for r in _read_csv(paths[1])
                  if r["Counter_Name"] == "GRBM_GUI_ACTIVE"
                  and _is_kernel(r["Kernel_Name"], kernel, args)) / 8
        busy = e.get("SQ_VALU_MFMA_BUSY_CYCLES", 0.0) / (cyc * 1024) if cyc else 0.0
        md.append(f"| {label} | {e['wps']} | {len(e['disp']) // 2} | "
                  f"{(e['SQ_INSTS_VALU'] - m) / m:.2f} | {e['SQ_INSTS_VALU_TRANS_F32'] / m:.2f} | "
                  f"{e['SQ_INSTS_LDS'] / m:.2f} | {e['SQ_INSTS_SALU'] / m:.2f} | {100 * busy:.1f}% | "
                  f"{100 * e['SQ_WAIT_ANY'] / wc:.1f}% | {100 * e['SQ_WAIT_INST_ANY'] / wc:.1f}% | "
                  f"{100 * e['SQ_ACTIVE_INST_VALU'] / wc:.1f}% | "
                  f"{100 * e['SQ_ACTIVE_INST_LDS'] / wc:.1f}% |")
    with open(os.path.join(prof, f"instruction_mix_{workload}.md"), "w") as f:
        f.write("\n".join(md) + "\n")


def _summarize_stored_ds(root, workload, w, shape, prof, cmd, ff, wf):
    """Kernel trace and HBM counters of the step with the backward through stored dS, when the
    three runs are there (trace, FETCH_SIZE, WRITE_SIZE of PROFILE_DS)."""
    tdir = os.path.join(root, "prof_trace_ds")
    if not os.path.isdir(tdir):
        return
    from paper_2507_16697_amd import ringx
    B, H, Nq, Nk, d, R = w.B, w.H, w.Nq, w.Nk, w.d, w.R
    stats = _read_csv(os.path.join(tdir, "ring8ds_kernel_stats.csv"))
    lines = []
    for r in stats:
        k = _profile_kernel(r["Name"])
        if k:
            lines.append((k[0], k[1], int(r["Calls"]), float(r["AverageNs"]), float(r["MinNs"]),
                          float(r["MaxNs"])))
    lines.sort(key=lambda x: -x[3] * x[2])
    slab = 2
    ds_slab = ringx.ringx_bwd_ds_bytes(H, H, Nq, Nk, d, R, slab)
    alg = {  # bytes per launch (one slab of two heads) that each kernel must move at least
        "bwd_dkdv_store": (2 * slab * Nk * d * 2 + 2 * slab * Nq * d * 2 + 2 * slab * Nq * 4,
                           ds_slab + 2 * slab * Nk * d * 4),
        "bwd_dq_ds": (ds_slab + slab * Nk * d * 2, slab * Nq * d * 4),
    }
    fetch = _pmc_per_dispatch(os.path.join(root, "pmc_ds_FETCH_SIZE"), "FETCH_SIZE") \
        if os.path.isdir(os.path.join(root, "pmc_ds_FETCH_SIZE")) else {}
    write = _pmc_per_dispatch(os.path.join(root, "pmc_ds_WRITE_SIZE"), "WRITE_SIZE") \
        if os.path.isdir(os.path.join(root, "pmc_ds_WRITE_SIZE")) else {}
    per = {}
    for src, which in ((fetch, 0), (write, 1)):
        for _, (name, val) in src.items():
            k = _profile_kernel(name)
            if k and k[1] in alg:
                per.setdefault(k[1], ([], []))[which].append(val)
    md = [f"# Backward through stored dS: {workload} ({shape})", "",
          "Commands (run from the repository root on one MI355X):", "",
          "    " + cmd("prof_trace_ds", "ring8ds", "--kernel-trace --stats") + PROFILE_DS,
          "    " + cmd("pmc_ds_FETCH_SIZE", "pmc", "--pmc FETCH_SIZE") + PROFILE_DS,
          "    " + cmd("pmc_ds_WRITE_SIZE", "pmc", "--pmc WRITE_SIZE") + PROFILE_DS, "",
          "Each run makes one plain step and two steps through stored dS (one untimed), each of "
          f"those a forward, a preprocess and {B * H // slab} slabs of {slab} heads (dK/dV with the "
          "dS stores, then dQ from the stored dS).  Durations in ns; only libringx kernels.", "",
          "| kernel | calls | average ns | min ns | max ns | total ms per step |",
          "|---|---|---|---|---|---|"]
    nsteps = {"bwd_dkdv_store": 2, "bwd_dq_ds": 2}
    for label, key, c, avg, mn, mx in lines:
        per_step = (c / nsteps[key] * avg / 1e6) if key in nsteps else float("nan")
        md.append(f"| {label} | {c} | {avg:.0f} | {mn:.0f} | {mx:.0f} | "
                  + (f"{per_step:.2f} |" if key in nsteps else "- |"))
    if per:
        md += ["", "HBM bytes per launch (one slab of two heads), counters calibrated as in "
               f"hbm_traffic_{workload}.md (fetched = FETCH_SIZE x 1024 x {ff:.4f}, written = "
               f"WRITE_SIZE x 1024 x {wf:.4f}), against the bytes the kernel must move:", "",
               "| kernel | fetched GB | algorithmic read GB | written GB | algorithmic write GB |",
               "|---|---|---|---|---|"]
        for key, (fv, wv) in per.items():
            fb = sorted(fv)[len(fv) // 2] * 1024 * ff if fv else float("nan")
            wb = sorted(wv)[len(wv) // 2] * 1024 * wf if wv else float("nan")
            md.append(f"| {key} | {fb / 1e9:.2f} | {alg[key][0] / 1e9:.2f} | {wb / 1e9:.2f} | "
                      f"{alg[key][1] / 1e9:.2f} |")
    with open(os.path.join(prof, f"kernel_trace_stored_ds_{workload}.md"), "w") as f:
        f.write("\n".join(md) + "\n")


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="ring8_nk262k_d128")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-rows", type=int, default=8192)
    ap.add_argument("--cpu-full", action="store_true",
                    help="also time the oracle on one full head of the workload and on the whole "
                         "16k single shard (minutes of host time)")
    ap.add_argument("--no-merge", action="store_true")
    ap.add_argument("--no-tokenizer", action="store_true",
                    help="skip the multi-fidelity tokenizer measurement (1024^3 x 4 field)")
    ap.add_argument("--no-gqa", action="store_true",
                    help="skip the grouped-query measurement (H/4 K/V heads)")
    ap.add_argument("--no-ring", action="store_true",
                    help="skip the ring-step measurement (chunks arriving on a second stream)")
    ap.add_argument("--no-stored-ds", action="store_true",
                    help="skip the step with the backward through stored dS")
    ap.add_argument("--no-shapes", action="store_true",
                    help="skip the other paper-shaped workloads (16k single shard, turbulence "
                         "tokens, 524k long step)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="only run a plain 1 GiB device-to-device copy (calibrates HBM byte counters)")
    ap.add_argument("--no-sclk", action="store_true",
                    help="do not sample the shader clock with rocm-smi (for runs under rocprofv3, "
                         "whose preloaded library would make the tool's own launcher initialise "
                         "the GPU)")
    ap.add_argument("--profile-summary", metavar="DIR",
                    help="CPU only: turn the rocprofv3 outputs under DIR (prof_trace, pmc_FETCH_SIZE, "
                         "pmc_WRITE_SIZE, pmc_copy_FETCH_SIZE, pmc_copy_WRITE_SIZE, pmc_busy; pmc_l2, pmc_stall1 "
                         "and pmc_stall2 when present) into "
                         "the summaries under profiles/")
    args = ap.parse_args()
    if args.profile_summary:
        summarize_profiles(args.profile_summary, args.workload)
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU's share of the ring; --gpus {args.gpus} is not supported "
              "(this build has no multi-GPU path)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_2507_16697_amd import inputs, ring, ringx

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(2)
    if args.copy_probe:
        src = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes_read": src.numel() * 4, "bytes_written": dst.numel() * 4,
                          "launches": 3}), flush=True)
        return
    w = inputs.WORKLOADS[args.workload]
    if w.dtype != "bf16" or w.passes != "fwd+bwd":
        print("bench.py times fwd+bwd bf16 workloads", file=sys.stderr)
        sys.exit(2)
    ringx.lib()  # fail loudly if the library is missing

    log(f"[bench] generating {w.name} inputs (seeded, host)")
    t0 = time.time()
    t = inputs.make_workload(w.name)
    log(f"[bench] inputs ready in {time.time() - t0:.1f}s; moving to HBM")
    sha = input_sha256(t)
    dev = torch.device("cuda:0")

    def to_dev(a):
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).to(dev).view(torch.bfloat16)

    q, k, v, do = (to_dev(t[n]) for n in ("q", "k", "v", "do"))
    B, H, Nq, Nk, d, R = w.B, w.H, w.Nq, w.Nk, w.d, w.R
    out = torch.empty_like(q)
    lse = torch.empty((B, H, Nq), dtype=torch.float32, device=dev)
    dq = torch.empty((B, H, Nq, d), dtype=torch.float32, device=dev)
    dk = torch.empty((B, H, Nk, d), dtype=torch.float32, device=dev)
    dv = torch.empty((B, H, Nk, d), dtype=torch.float32, device=dev)
    ws = torch.empty(ringx.ringx_bwd_workspace_bytes(B, H, Nq, Nk, d, R, ringx.RINGX_BF16),
                     dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream()

    delta = ws[: 2 * B * H * Nq * 4].view(torch.float32).view(2, B, H, Nq)

    def step(ev=None):
        # one step = ringx_attn_fwd + ringx_attn_bwd; the backward is issued as its three stages
        # (exactly what ringx_attn_bwd enqueues) so that each kernel gets its own event pair
        marks = ev or [None] * 5
        if marks[0]: marks[0].record(stream)
        ringx.ringx_attn_fwd(q, k, v, R, scale=w.scale, out=out, lse=lse, stream=stream)
        if marks[1]: marks[1].record(stream)
        ringx.ringx_bwd_preprocess(out, do, lse, delta=delta, stream=stream)
        if marks[2]: marks[2].record(stream)
        ringx.ringx_attn_bwd_dkdv(q, k, v, do, lse, delta, R, scale=w.scale, dk=dk, dv=dv,
                                  stream=stream)
        if marks[3]: marks[3].record(stream)
        ringx.ringx_attn_bwd_dq(q, k, v, do, lse, delta, R, scale=w.scale, dq=dq, stream=stream)
        if marks[4]: marks[4].record(stream)

    for i in range(args.warmup):
        step()
        torch.cuda.synchronize()
        log(f"[bench] warmup step {i + 1}/{args.warmup} done")

    K = args.steps
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(5)] for _ in range(K)]
    torch.cuda.synchronize()
    with ClockSampler(enabled=not args.no_sclk) as clock:
        wall0 = time.perf_counter()
        for s_ in range(K):
            step(ev[s_])
        torch.cuda.synchronize()
        wall = time.perf_counter() - wall0
    total_ms = ev[0][0].elapsed_time(ev[K - 1][4])

    def avg(i, j):
        return sum(e[i].elapsed_time(e[j]) for e in ev) / K

    fwd_ms, pre_ms, dkdv_ms, dq_ms = avg(0, 1), avg(1, 2), avg(2, 3), avg(3, 4)
    bwd_ms = pre_ms + dkdv_ms + dq_ms
    ms_step = total_ms / K
    per_step = sorted(e[0].elapsed_time(e[4]) for e in ev)
    log(f"[bench] timed {K} steps: {ms_step:.2f} ms/step (fwd {fwd_ms:.2f}, bwd {bwd_ms:.2f} = "
        f"pre {pre_ms:.3f} + dkdv {dkdv_ms:.2f} + dq {dq_ms:.2f}; wall {wall * 1e3 / K:.2f})")
    if not (torch.isfinite(out.float()).all() and torch.isfinite(dq).all()):
        raise RuntimeError("non-finite results")
    dq_step = dq.clone()      # the other measurements below reuse dq

    U = w.gemm_unit()                      # 2*B*H*Nq*Nk*d
    value = 6 * U / (ms_step * 1e-3) / 1e12

    def tf(flops, ms):
        return flops / (ms * 1e-3) / 1e12

    kernels = {
        "fwd_bf16_kernel": {"ms": fwd_ms, "flops": 2 * U, "work": "4*B*H*Nq*Nk*d (QK^T, PV)",
                            "tflops": tf(2 * U, fwd_ms),
                            "traffic": load_traffic("fwd_bf16", w.name,
                                                    kernel_source_hash(["fwd_bf16.hip", "ringx_device.h"]))},
        # the backward's four algorithmic contractions (dV, dP, dK, dQ) are credited to the kernel
        # that computes them first: dP is part of the dK/dV pass, the dQ pass recomputes S and dP
        "bwd_dkdv_kernel": {"ms": dkdv_ms, "flops": 3 * U,
                            "work": "6*B*H*Nq*Nk*d credited (dV, dP, dK); S recomputed",
                            "tflops": tf(3 * U, dkdv_ms),
                            "traffic": load_traffic("bwd_dkdv", w.name,
                                                    kernel_source_hash(["bwd_bf16.hip", "ringx_device.h"]))},
        "bwd_dq_kernel": {"ms": dq_ms, "flops": U,
                          "work": "2*B*H*Nq*Nk*d credited (dQ); S and dP recomputed",
                          "tflops": tf(U, dq_ms),
                          "traffic": load_traffic("bwd_dq", w.name,
                                                  kernel_source_hash(["bwd_dq_bf16.hip", "ringx_device.h"]))},
        # reads out, dout (bf16) and lse; writes D and nl
        "bwd_pre_bf16_kernel": {"ms": pre_ms, "bytes": B * H * Nq * (4 * d + 12),
                                "GB/s": B * H * Nq * (4 * d + 12) / (pre_ms * 1e-3) / 1e9},
    }
    # executed products (the recomputed S and dP included): what the matrix cores actually ran
    for name, units in (("fwd_bf16_kernel", 2), ("bwd_dkdv_kernel", 4), ("bwd_dq_kernel", 3)):
        kernels[name]["frac"] = kernels[name]["tflops"] / PEAK_BF16_TFLOPS
        kernels[name]["executed_flops"] = units * U
        kernels[name]["executed_tflops"] = tf(units * U, kernels[name]["ms"])
        kernels[name]["executed_frac"] = kernels[name]["executed_tflops"] / PEAK_BF16_TFLOPS
    dominant = max(("fwd_bf16_kernel", "bwd_dkdv_kernel", "bwd_dq_kernel"),
                   key=lambda n: kernels[n]["ms"])
    dom = kernels[dominant]
    roofline = {
        "kernel": dominant, "bound": "mfma", "achieved": dom["tflops"], "peak": PEAK_BF16_TFLOPS,
        "unit": "TFLOP/s", "frac": dom["frac"], "traffic": dom["traffic"],
        "work_per_launch": f"{dom['flops']:.4e} flops = {dom['work']}",
        # one call of ringx_attn_bwd_dkdv runs its kernel on groups of K/V heads of about 16 rounds
        # of 256 workgroups each (two heads at the 8-way ring share)
        "dispatches_per_call": _dkdv_dispatches(B * H, Nk, R) if dominant == "bwd_dkdv_kernel" else 1,
    }

    # standalone Eq. (5) merge of the R per-chunk partials (an HBM-bound kernel)
    if not args.no_merge:
        part_out, part_lse = ringx.ringx_attn_fwd_partials(q, k, v, R, scale=w.scale, stream=stream)
        mo = torch.empty_like(q)
        ml = torch.empty_like(lse)
        ringx.ringx_lse_merge(part_out, part_lse, out=mo, lse=ml, stream=stream)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        nm = 10
        e0.record(stream)
        for _ in range(nm):
            ringx.ringx_lse_merge(part_out, part_lse, out=mo, lse=ml, stream=stream)
        e1.record(stream)
        torch.cuda.synchronize()
        mms = e0.elapsed_time(e1) / nm
        rows = B * H * Nq
        mbytes = R * rows * (4 * d + 4) + rows * (2 * d + 4)
        kernels["lse_merge"] = {"ms": mms, "bytes": mbytes, "GB/s": mbytes / (mms * 1e-3) / 1e9,
                                "frac": mbytes / (mms * 1e-3) / 1e9 / PEAK_HBM_GBS,
                                "traffic": load_traffic("lse_merge", w.name,
                                                        kernel_source_hash(["merge.hip", "ringx_device.h"]))}
        log(f"[bench] lse_merge {mms:.3f} ms, {kernels['lse_merge']['GB/s']:.0f} GB/s")
        del part_out, part_lse

    # the same step as R ring steps: every chunk arrives in a ping-pong buffer by a device copy on
    # a second stream while the previous chunk is computed (ringx_attn_fwd_step / _bwd_step)
    if not args.no_ring:
        bounds = [ringx.ringx_chunk_bounds(Nk, R, r) for r in range(R)]
        ks = [k[:, :, lo:hi].contiguous() for lo, hi in bounds]
        vs = [v[:, :, lo:hi].contiguous() for lo, hi in bounds]

        def ring_step():
            o, l = ring.ring_forward(q, ks, vs, scale=w.scale)
            ring.ring_backward(q, ks, vs, o, do, l, scale=w.scale)

        ring_step()
        torch.cuda.synchronize()
        nr = max(1, min(K, 3))
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(nr):
            ring_step()
        e1.record(stream)
        torch.cuda.synchronize()
        rms = e0.elapsed_time(e1) / nr
        kernels["ring_steps"] = {
            "ms": rms, "steps": nr, "chunks": R,
            "tflops": 6 * U / (rms * 1e-3) / 1e12,
            "overhead_vs_fused": rms / ms_step - 1.0,
            "copied_bytes": 2 * B * H * Nk * d * 2 * 2,
            "what": "fwd+bwd as R ring steps, chunk copies overlapped on a second stream",
        }
        log(f"[bench] ring steps: {rms:.2f} ms/step ({100 * (rms / ms_step - 1):+.1f}% vs fused)")
        del ks, vs

    # grouped-query attention on the same shapes: H/4 K/V heads (the first H/4 heads of K and V)
    if not args.no_gqa and H % 4 == 0:
        hkv = H // 4
        kg, vg = k[:, :hkv].contiguous(), v[:, :hkv].contiguous()
        dkg = torch.empty((B, hkv, Nk, d), dtype=torch.float32, device=dev)
        dvg = torch.empty_like(dkg)

        def gqa_step():
            o, l = ringx.ringx_attn_fwd_gqa(q, kg, vg, R, scale=w.scale, out=out, lse=lse,
                                            stream=stream)
            ringx.ringx_attn_bwd_gqa(q, kg, vg, o, do, l, R, scale=w.scale, dq=dq, dk=dkg,
                                     dv=dvg, stream=stream)

        gqa_step()
        torch.cuda.synchronize()
        ng = max(1, min(K, 3))
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(ng):
            gqa_step()
        e1.record(stream)
        torch.cuda.synchronize()
        gms = e0.elapsed_time(e1) / ng
        kernels["gqa_steps"] = {"ms": gms, "steps": ng, "H": H, "Hkv": hkv,
                                "tflops": 6 * U / (gms * 1e-3) / 1e12,
                                "what": "fwd+bwd with H/4 K/V heads (grouped-query attention)"}
        log(f"[bench] gqa (Hkv={hkv}): {gms:.2f} ms/step, {6 * U / (gms * 1e-3) / 1e12:.1f} TFLOP/s")
        del kg, vg, dkg, dvg

    # the same step with the backward through stored dS (ringx_attn_bwd_ds as its stages): the
    # dK/dV kernel also writes every bf16 dS, and dQ is streamed from them (7U executed instead of
    # 9U), in slabs of two K/V heads (2 B H Nq Nk / (B H) * 2 bytes of workspace)
    ds_need = ringx.ringx_bwd_ds_bytes(H, H, Nq, Nk, d, R, 2) if d == 128 and B * H >= 2 else 0
    ds_fits = ds_need > 0 and torch.cuda.mem_get_info(dev)[0] > ds_need + (4 << 30)
    if not args.no_stored_ds and ds_need and not ds_fits:
        log(f"[bench] stored dS skipped: {ds_need / 2**30:.0f} GiB of workspace does not fit")
    if not args.no_stored_ds and ds_fits:
        slab = 2
        ds_buf = torch.empty(ds_need, dtype=torch.uint8, device=dev)
        dq_s = torch.empty_like(dq)
        nslab = (B * H + slab - 1) // slab

        def stored_step(marks=None):
            m = marks or [None] * (2 + 2 * nslab)
            if m[0]: m[0].record(stream)
            ringx.ringx_attn_fwd(q, k, v, R, scale=w.scale, out=out, lse=lse, stream=stream)
            ringx.ringx_bwd_preprocess(out, do, lse, delta=delta, stream=stream)
            for i in range(nslab):
                kv0, n = i * slab, min(slab, B * H - i * slab)
                if m[1 + 2 * i]: m[1 + 2 * i].record(stream)
                ringx.ringx_attn_bwd_dkdv_ds(q, k, v, do, lse, delta, R, ds_buf, kv0, n,
                                             scale=w.scale, dk=dk, dv=dv, stream=stream)
                if m[2 + 2 * i]: m[2 + 2 * i].record(stream)
                ringx.ringx_attn_bwd_dq_ds(ds_buf, k, (B, H, Nq, d), R, kv0, n, scale=w.scale,
                                           dq=dq_s, stream=stream)
            if m[-1]: m[-1].record(stream)

        stored_step()
        torch.cuda.synchronize()
        ns = max(1, min(K, 3))
        evs = [[torch.cuda.Event(enable_timing=True) for _ in range(2 + 2 * nslab)]
               for _ in range(ns)]
        for i in range(ns):
            stored_step(evs[i])
        torch.cuda.synchronize()
        sms = sum(e[0].elapsed_time(e[-1]) for e in evs) / ns
        s_dkdv = sum(e[1 + 2 * i].elapsed_time(e[2 + 2 * i]) for e in evs
                     for i in range(nslab)) / ns
        s_dq = sum(e[2 + 2 * i].elapsed_time(e[3 + 2 * i] if 3 + 2 * i < len(e) - 1 else e[-1])
                   for e in evs for i in range(nslab)) / ns
        ds_total = ringx.ringx_bwd_ds_bytes(H, H, Nq, Nk, d, R, B * H)
        # the dQ pass reads every stored dS once, K once per head, and writes dq
        dq_bytes = ds_total + B * H * Nk * d * 2 + B * H * Nq * d * 4
        kernels["stored_ds_steps"] = {
            "ms": sms, "steps": ns, "slab_heads": slab, "workspace_bytes": int(ds_buf.numel()),
            "tflops": 6 * U / (sms * 1e-3) / 1e12,
            "vs_recompute_step": sms / ms_step - 1.0,
            "bwd_dkdv_kernel_store": {"ms": s_dkdv, "executed_tflops": tf(4 * U, s_dkdv),
                                      "ds_bytes_written": ds_total,
                                      "GB/s_written": ds_total / (s_dkdv * 1e-3) / 1e9},
            "bwd_dq_ds_kernel": {"ms": s_dq, "bytes": dq_bytes, "executed_tflops": tf(U, s_dq),
                                 "GB/s": dq_bytes / (s_dq * 1e-3) / 1e9,
                                 "frac": dq_bytes / (s_dq * 1e-3) / 1e9 / PEAK_HBM_GBS},
            "what": "fwd + bwd with dS stored by the dK/dV pass and dQ streamed from it "
                    "(7U of matrix products executed instead of 9U)",
        }
        rq = float(((dq_s - dq_step).double().pow(2).mean().sqrt() /
                    dq_step.double().pow(2).mean().sqrt()))
        kernels["stored_ds_steps"]["dq_rel_rms_vs_recompute"] = rq
        log(f"[bench] stored dS: {sms:.2f} ms/step ({100 * (sms / ms_step - 1):+.1f}% vs recompute;"
            f" dkdv+store {s_dkdv:.2f}, dq from dS {s_dq:.2f} ms = "
            f"{dq_bytes / (s_dq * 1e-3) / 1e12:.2f} TB/s)")
        del ds_buf, dq_s

    # multi-fidelity tokenizer: the three fidelity modes of Table III's (filter, ratio) pairs
    # (1, 8x), (4, 2x), (8, 1x) with patch 1 over a DNS-sized 1024^3 x 4 fp32 field
    if not args.no_tokenizer:
        gen = torch.Generator(device=dev)
        gen.manual_seed(7)
        C_, D_ = 4, 1024
        field = torch.randn((C_, D_, D_, D_), device=dev, generator=gen)
        def time_modes(centre):
            modes = []
            for k_, ratio in ((1, 8), (4, 2), (8, 1)):
                tok = ringx.ringx_tt_tokenize(field, k_, ratio, centre, 1, stream=stream)
                torch.cuda.synchronize()
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                # the (1, 8x) crop runs for about 14 us, less than the binding takes to enqueue a
                # call: a spin kernel holds the stream until all calls are queued, so that the
                # events time the kernels back to back rather than the host's launch rate
                torch.cuda._sleep(20_000_000)
                e0.record(stream)
                for _ in range(20):
                    ringx.ringx_tt_tokenize(field, k_, ratio, centre, 1, tokens=tok, stream=stream)
                e1.record(stream)
                torch.cuda.synchronize()
                tms = e0.elapsed_time(e1) / 20
                nbytes = C_ * (D_ // ratio) ** 3 * 4 + tok.numel() * 4
                modes.append({"filter": k_, "ratio": ratio, "tokens": tok.shape[0], "ms": tms,
                              "bytes": nbytes, "GB/s": nbytes / (tms * 1e-3) / 1e9,
                              "frac": nbytes / (tms * 1e-3) / 1e9 / PEAK_HBM_GBS})
                del tok
            return modes

        # subdomains starting on a 16-byte boundary along x, and one cell off it (three of four
        # crop centres)
        modes = time_modes((D_ // 2, D_ // 3, D_ // 5))
        modes_off = time_modes((D_ // 2, D_ // 3, D_ // 5 + 1))
        kernels["tt_tokenize"] = {"field": f"{C_}x{D_}^3 fp32", "patch": 1, "modes": modes,
                                  "modes_misaligned": modes_off, "bound": "hbm"}
        for lab, ms_ in (("aligned", modes), ("misaligned", modes_off)):
            log(f"[bench] tokenizer, {lab} subdomain: " + ", ".join(
                f"(k={m['filter']}, {m['ratio']}x) {m['ms']:.3f} ms {m['GB/s']:.0f} GB/s" for m in ms_))
        del field

    # the other paper-shaped workloads (parity-test cases, reported beside the headline)
    if not args.no_shapes:
        del out, dq, dk, dv
        kernels["other_shapes"] = other_shapes(torch, np, inputs, ringx, stream, dev)

    result = {
        "metric": METRIC, "value": value, "unit": "TFLOP/s", "n_gpus": 1, "steps": K,
        "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": w.name, "B": B, "H": H, "Nq": Nq, "Nk": Nk, "d": d, "R": R,
                   "flops_per_step": 6 * U, "flop_convention": "12*B*H*Nq*Nk*d per fwd+bwd step",
                   "fwd_ms": fwd_ms, "bwd_ms": bwd_ms, "bwd_pre_ms": pre_ms,
                   "bwd_dkdv_ms": dkdv_ms, "bwd_dq_ms": dq_ms,
                   "step_ms_min": per_step[0], "step_ms_median": per_step[len(per_step) // 2],
                   "step_ms_max": per_step[-1],
                   "tflops_fa_convention_14": 7 * U / (ms_step * 1e-3) / 1e12},
        "pct_of_peak": 100.0 * value / PEAK_BF16_TFLOPS,
        "roofline": roofline,
        "kernels": kernels,
        "gpu": torch.cuda.get_device_name(0),
        "hip": torch.version.hip,
        "sclk": clock.record(),
        "inputs": {"recipe": f"seeded host generator, {w.name} (per-slab PCG64 streams)",
                   "sha256": sha},
        # the paper's own figures, system-level on other hardware: context, not a target (the
        # paper reports no single-GPU throughput for this kernel path, so vs_baseline is null)
        "paper_context": {
            "sustained": "1.1 EFLOPS (attention flops, Eq. (7)) on 32,768 MI250X GCDs of Frontier, "
                         "about 33.6 TFLOP/s per GCD, mixed fp32-bf16",
            "scaling": "94% weak-scaling efficiency from 256 to 32,768 GCDs",
        },
    }
    if not args.no_cpu_baseline:
        log(f"[bench] cpu baseline: oracle on {args.cpu_rows} query rows of head 0")
        result["cpu_baseline"] = cpu_baseline(t, w, args.cpu_rows, full_head=args.cpu_full)
        log(f"[bench] cpu baseline {result['cpu_baseline']['seconds']:.1f}s")
    else:
        result["cpu_baseline"] = None
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
