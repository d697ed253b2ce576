#!/usr/bin/env python3
"""Benchmark of the PSKV hot path on one MI355X.

A "step" is one pskv_attn_fwd call: the whole per-layer hot path (stack the suffix queries,
prefix scores/values on the matrix cores, causal suffix part, online-softmax combine, store)
over one batch of B synthetic candidates, with every tensor resident in HBM before timing.
The default workload is the 8B-class GQA shape on which the throughput goal is stated.

Prints ONE JSON line.  `value` = candidate suffixes per second per attention layer.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0     # MI355X dense bf16 MFMA
PEAK_F64_TFLOPS = 78.6        # MI355X fp64 vector
PEAK_HBM_GBS = 8000.0         # MI355X HBM3E
PRERAMP_LAUNCHES = 300        # untimed launches right before the counted warm-up: the shader clock
                              # climbs from idle over roughly the first hundred launches of a run


FORWARD_SOURCES = ("pskv_internal.h", "pskv_mfma.hpp", "pskv_packed.hpp", "pskv_resident.hip", "pskv_stream.hip", "pskv_simple.hip")
BACKWARD_SOURCES = FORWARD_SOURCES + ("pskv_bwd_mfma.hip", "pskv_bwd_simple.hip")


def kernel_source_rev(files=FORWARD_SOURCES) -> str:
    """Short hash of the kernel sources a set of offline counter readings is tied to (the forward
    kernels' files for the forward table, those plus the backward kernels' for the backward table)."""
    import hashlib
    csrc = os.path.join(ROOT, "paper_2603_13420_amd", "csrc")
    h = hashlib.sha1()
    for f in files:
        h.update(open(os.path.join(csrc, f), "rb").read())
    return h.hexdigest()[:12]


def offline_counters(table, name, impl_auto: bool, files=FORWARD_SOURCES):
    """(traffic bytes, executed matrix-core flops, source note) from the offline rocprofv3 readings of
    `name`, or Nones with the reason when there are none or the kernels have changed since."""
    tr = table.get(name) if impl_auto else None
    if tr is None:
        return None, None, "no offline rocprofv3 reading for this configuration"
    rev = kernel_source_rev(files)
    if tr.get("rev") != rev:
        return None, None, (f"stale: {tr['file']} was measured on kernel sources {tr.get('rev')}, these are {rev}; "
                            "collect it again (the command is in that file)")
    traffic = (tr["fetch_kib"] * tr["fetch_scale"] + tr["write_kib"] * tr["write_scale"]) * 1024
    return traffic, tr.get("mfma_flops"), f"offline: profiles/{tr['file']} (rocprofv3 --pmc, kernel sources {rev})"


def alg_counts(w, suf_len, pre_len=None):
    """Algorithmic work of one call: multiply-adds over visible keys only at 2 FLOP each, and
    the bytes that must cross HBM once (valid Q rows in, valid O rows out, valid suffix K/V
    rows in, every real prefix K/V row once).  pre_len: real prefix rows per instruction of
    the multi-instruction form (None: one shared prefix of w.P rows)."""
    import numpy as np
    l = suf_len.astype(np.int64)
    e = 2 if w.dtype == "bf16" else 4
    if pre_len is None:
        P, prefix_rows = w.P, w.P
    else:
        P = np.repeat(pre_len.astype(np.int64), w.C)      # the candidate's own prefix length
        prefix_rows = int(pre_len.astype(np.int64).sum())
    flops = int((w.Hq * 4 * w.D * (l * P + l * (l + 1) // 2)).sum())
    exps = int((w.Hq * (l * P + l * (l + 1) // 2)).sum())
    prefix_bytes = 2 * prefix_rows * w.Hkv * w.D * e
    bytes_ = int(l.sum()) * (2 * w.Hq + 2 * w.Hkv) * w.D * e + prefix_bytes
    return flops, bytes_, prefix_bytes, exps


# HBM traffic of one launch as read by rocprofv3 (FETCH_SIZE / WRITE_SIZE, KiB per dispatch), with
# the factor by which the same counter under- or over-reads a plain copy kernel of known size, and
# the matrix-core work the launch executes (SQ_INSTS_VALU_MFMA_MOPS_BF16 * 512 flop, whole tiles).
# OFFLINE measurements: commands and raw readings are in profiles/<file>; "rev" is the hash of the
# kernel sources they were taken on (kernel_source_rev()).  When the sources have changed since, the
# bench line reports no traffic and says why, instead of a figure that no longer holds.
HBM_TRAFFIC = {
    "gqa8b_bf16": {"file": "resident_packed_kernel_gqa8b_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 96901005312.0, "fetch_kib": 159093.8, "fetch_scale": 2.0, "write_kib": 196608.6, "write_scale": 1.0},
    "ldec_gqa8b_bf16": {"file": "stream_candidate4_kernel_ldec_gqa8b_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 134809124864.0, "fetch_kib": 224501.7, "fetch_scale": 2.0, "write_kib": 327680.0, "write_scale": 1.0},
    "ldec_qwen7b_bf16": {"file": "stream_candidate4_kernel_ldec_qwen7b_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 116735868928.0, "fetch_kib": 168966.7, "fetch_scale": 2.0, "write_kib": 286720.0, "write_scale": 1.0},
    "longprefix_bf16": {"file": "stream_pipelined_kernel_longprefix_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 279172874240.0, "fetch_kib": 63775.3, "fetch_scale": 2.0, "write_kib": 66570.0, "write_scale": 1.0},
    "mha13b_bf16": {"file": "stream_packed_kernel_mha13b_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 2351263907840.0, "fetch_kib": 3070860.5, "fetch_scale": 2.0, "write_kib": 2621441.3, "write_scale": 1.0},
    "mha7b_bf16": {"file": "resident_packed_kernel_mha7b_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 42949672960.0, "fetch_kib": 124703.9, "fetch_scale": 2.0, "write_kib": 82075.1, "write_scale": 1.0},
    "multi32_gqa8b_bf16": {"file": "resident_packed_kernel_multi32_gqa8b_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 74151100416.0, "fetch_kib": 167936.0, "fetch_scale": 2.0, "write_kib": 196611.6, "write_scale": 1.0},
    "multi4_long_bf16": {"file": "stream_pipelined_kernel_multi4_long_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 73014444032.0, "fetch_kib": 53987.6, "fetch_scale": 2.0, "write_kib": 66593.5, "write_scale": 1.0},
    "multi8_gqa8b_bf16": {"file": "resident_packed_kernel_multi8_gqa8b_bf16_hbm_traffic.txt", "rev": "f5f190b7a8cd", "mfma_flops": 80480305152.0, "fetch_kib": 159080.0, "fetch_scale": 2.0, "write_kib": 196608.9, "write_scale": 1.0},
}


def cpu_baseline(inp, budget_s=12.0):
    """Time the CPU oracle, as it stands, on a bounded sample of the same workload."""
    import numpy as np
    from oracle import pskv_oracle as orc
    w = inp.w
    n = min(w.B, 8)
    t_total, done = 0.0, 0
    # grow the sample until roughly budget_s seconds of oracle time have been spent,
    # wrapping round the batch when the whole workload takes less than that
    while t_total < budget_s:
        first = done % w.B
        n = min(n, w.B - first)
        sub = inp.take(np.arange(first, first + n))
        t0 = time.perf_counter()
        orc.attn(sub.q, sub.k_suf, sub.v_suf, sub.k_pre, sub.v_pre, sub.suf_len, sub.scale, w.dtype)
        t_total += time.perf_counter() - t0
        done += n
        rate = done / t_total
        n = int(max(1, min(w.B, rate * max(budget_s - t_total, 0.0) / 2 + 1)))
    return {"value": done / t_total, "unit": "candidates/s", "cores": orc.threads(), "kind": "oracle",
            "sample": f"{done} candidates (the {w.B} of {w.name} taken in order, wrapping round; all heads), "
                      f"{t_total:.1f} s of oracle time"}


def cpu_baseline_multi(inp, budget_s=12.0):
    """The multi-instruction oracle timed on whole instructions of the same workload, in order."""
    import numpy as np
    from oracle import pskv_oracle as orc
    w = inp.w
    t_total, done, n = 0.0, 0, 0
    while t_total < budget_s:
        sub = inp.take_instructions(np.array([n % w.Np]))
        t0 = time.perf_counter()
        orc.attn_multi(sub.q, sub.k_suf, sub.v_suf, sub.k_pre, sub.v_pre, sub.pre_len, sub.suf_len, sub.scale, w.dtype)
        t_total += time.perf_counter() - t0
        done += w.C
        n += 1
    return {"value": done / t_total, "unit": "candidates/s", "cores": orc.threads(), "kind": "oracle",
            "sample": f"{n} instructions with their {w.C} candidates each (those of {w.name} in order, wrapping "
                      f"round; all heads), {t_total:.1f} s of oracle time"}


# The same for one backward call (its two kernels together).
HBM_TRAFFIC_BWD = {
    "gqa8b_bf16": {"file": "bwd_kernels_gqa8b_bf16_hbm_traffic.txt", "rev": "479d58512a69", "mfma_flops": 170215342080.0, "fetch_kib": 548682.5, "fetch_scale": 2.0, "write_kib": 297876.7, "write_scale": 1.0},
    "ldec_gqa8b_bf16": {"file": "bwd_kernels_ldec_gqa8b_bf16_hbm_traffic.txt", "rev": "479d58512a69", "mfma_flops": 313824116736.0, "fetch_kib": 904869.2, "fetch_scale": 2.0, "write_kib": 496137.1, "write_scale": 1.0},
    "longprefix_bf16": {"file": "bwd_kernels_longprefix_bf16_hbm_traffic.txt", "rev": "479d58512a69", "mfma_flops": 427349245952.0, "fetch_kib": 216717.6, "fetch_scale": 2.0, "write_kib": 99366.9, "write_scale": 1.0},
    "mha7b_bf16": {"file": "bwd_kernels_mha7b_bf16_hbm_traffic.txt", "rev": "479d58512a69", "mfma_flops": 81604378624.0, "fetch_kib": 374563.8, "fetch_scale": 2.0, "write_kib": 247297.4, "write_scale": 1.0},
}


def bench_backward(args):
    """One step = one pskv_attn_bwd call (gradients with respect to q, k_suf, v_suf from out, lse
    and dout, everything resident in HBM).  Prints one JSON line of the same form."""
    import numpy as np
    import torch
    from paper_2603_13420_amd import binding as pk, inputs as gen
    from oracle import parity
    w = gen.WORKLOADS[args.workload]
    inp = gen.make_inputs(w, pad="zero", workers=16)
    l = inp.suf_len.astype(np.int64)
    e = 2 if w.dtype == "bf16" else 4
    vis_pre, vis_suf = int((l * w.P).sum()), int((l * (l + 1) // 2).sum())
    # s and dp once per visible pair, then dq (all pairs), dk and dv (suffix pairs): 2 flop per multiply-add
    flops = w.Hq * 2 * w.D * (3 * vis_pre + 5 * vis_suf)
    bytes_ = int(l.sum()) * (4 * w.Hq + 4 * w.Hkv) * w.D * e + int(l.sum()) * w.Hq * 4 + 2 * w.P * w.Hkv * w.D * e
    nsets = args.sets or 2
    base = gen.to_device(inp)
    dout_host, dout64 = gen.make_dout(inp, w.seed + 7)
    dout0 = (torch.from_numpy(dout_host).view(torch.bfloat16) if w.dtype == "bf16" else torch.from_numpy(dout_host)).to("cuda:0")
    dout0 = torch.nan_to_num(dout0, nan=0.0)
    sets = []
    for s_ in range(nsets):
        d = base if s_ == 0 else {k: (v.clone() if k in ("q", "k_suf", "v_suf") else v) for k, v in base.items()}
        lse = torch.empty((w.B, w.Hq, w.S), dtype=torch.float32, device="cuda:0")
        out = pk.pskv_attn_fwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], lse=lse,
                               scale=inp.scale)
        sets.append(dict(d, out=out, lse=lse, dout=dout0.clone(), dq=torch.empty_like(d["q"]),
                         dk=torch.empty_like(d["k_suf"]), dv=torch.empty_like(d["k_suf"]),
                         ws=torch.empty(w.B * w.Hq * w.S * 4, dtype=torch.uint8, device="cuda:0")))
    torch.cuda.synchronize()

    def call(i):
        d = sets[i]
        pk.pskv_attn_bwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], d["out"], d["lse"],
                         d["dout"], dq=d["dq"], dk_suf=d["dk"], dv_suf=d["dv"], impl=args.impl, scale=inp.scale,
                         workspace=d["ws"])

    steps, warmup = min(args.steps, 400), min(args.warmup, 100)
    for i in range(args.preramp // 2 + warmup):      # clock ramp (untimed, fixed), then the counted warm-up
        call(i % nsets)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    ev0.record()
    for i in range(steps):
        call(i % nsets)
    ev1.record()
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t0) * 1e3 / steps
    kern_ms = ev0.elapsed_time(ev1) / steps
    cand = np.array([0, w.B - 1])
    sub = inp.take(cand)
    rq, rk, rv = parity.oracle_bwd(sub, dout64[cand])
    sel = torch.from_numpy(cand).to("cuda:0")
    valid = np.arange(w.S)[None, :] < sub.suf_len[:, None]
    chk = {n: parity.compare_grad(gen.out_to_f64(sets[0][key][sel]), r, valid, w.dtype, f"bench self-check {n}")
           for n, key, r in (("dq", "dq", rq), ("dk_suf", "dk", rk), ("dv_suf", "dv", rv))}
    mfma = w.dtype == "bf16" and args.impl != "simple"
    compute = {"bound": "mfma" if mfma else "alu", "achieved": flops / (kern_ms * 1e-3) / 1e12,
               "peak": PEAK_BF16_TFLOPS if mfma else (PEAK_F64_TFLOPS if w.dtype == "f32" else 157.3), "unit": "TFLOP/s",
               "alg_flops_per_step": flops}
    compute["frac"] = compute["achieved"] / compute["peak"]
    hbm = {"bound": "hbm", "achieved": bytes_ / (kern_ms * 1e-3) / 1e9, "peak": PEAK_HBM_GBS, "unit": "GB/s",
           "alg_bytes_per_step": bytes_}
    hbm["frac"] = hbm["achieved"] / hbm["peak"]
    roof, other = (hbm, compute) if bytes_ / (PEAK_HBM_GBS * 1e9) >= flops / (compute["peak"] * 1e12) else (compute, hbm)
    roof["traffic"], _, roof["traffic_source"] = offline_counters(HBM_TRAFFIC_BWD, w.name, args.impl == "auto", BACKWARD_SOURCES)
    roof["traffic_unit"] = "bytes per step"
    roof["kernel_ms"] = kern_ms
    line = {"metric": "candidate suffixes/sec per attention layer, backward pass", "value": w.B / (ms_per_step * 1e-3),
            "unit": "candidates/s", "n_gpus": 1, "steps": steps, "warmup": warmup, "preramp_launches": args.preramp // 2,
            "ms_per_step": ms_per_step,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "bf16" if mfma else ("f64" if w.dtype == "f32" else "f32"), "data": "synthetic",
            "config": {"workload": w.name, "pass": "backward", "B": w.B, "P": w.P, "S": w.S,
                       "suffix_len": [w.len_lo, w.len_hi], "Hq": w.Hq, "Hkv": w.Hkv, "D": w.D, "impl": args.impl,
                       "buffer_sets": nsets, "seed": w.seed},
            "roofline": roof, "roofline_" + other["bound"]: other, "self_check": chk}
    if not args.no_cpu_baseline:
        from oracle import pskv_oracle as orc
        t_total, done, n = 0.0, 0, 4
        while t_total < 12.0:
            first = done % w.B
            n = min(n, w.B - first)
            c = np.arange(first, first + n)
            sb = inp.take(c)
            t1 = time.perf_counter()
            orc.attn_bwd(sb.q, sb.k_suf, sb.v_suf, sb.k_pre, sb.v_pre, sb.suf_len, np.nan_to_num(dout64[c]), sb.scale, w.dtype)
            t_total += time.perf_counter() - t1
            done += n
            n = int(max(1, min(w.B, done / t_total * max(12.0 - t_total, 0.0) / 2 + 1)))
        line["cpu_baseline"] = {"value": done / t_total, "unit": "candidates/s", "cores": orc.threads(), "kind": "oracle",
                                "sample": f"{done} candidates of {w.name} in order (wrapping round), backward oracle, "
                                          f"{t_total:.1f} s"}
    print(json.dumps(line), flush=True)


def measure_mfma_peak(torch, stream) -> float:
    """What the matrix cores of this machine sustain with nothing else going on (TFLOP/s): the MFMA-only
    kernel of libpskv_probe.so, a few launches to let the clock settle, then a timed one."""
    import ctypes
    path = os.path.join(ROOT, "paper_2603_13420_amd", "libpskv_probe.so")
    if not os.path.exists(path):
        return float("nan")
    lib = ctypes.CDLL(path)
    lib.pskv_probe_mfma_launch.restype = ctypes.c_int
    lib.pskv_probe_mfma_launch.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_double)]
    sink = torch.zeros(1, dtype=torch.float32, device="cuda:0")
    flops = ctypes.c_double(0.0)
    iters = 500         # 0.2 ms per launch

    def launch():
        rc = lib.pskv_probe_mfma_launch(iters, ctypes.c_void_p(sink.data_ptr()), ctypes.c_void_p(stream), ctypes.byref(flops))
        assert rc == 0, f"probe launch failed with HIP status {rc}"

    for _ in range(100):
        launch()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(200):
        launch()
    e1.record()
    e1.synchronize()
    return flops.value * 200 / (e0.elapsed_time(e1) * 1e-3) / 1e12


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2000)
    ap.add_argument("--warmup", type=int, default=500)
    ap.add_argument("--workload", default="gqa8b_bf16")
    ap.add_argument("--impl", default="auto")
    ap.add_argument("--sets", type=int, default=0, help="rotating input/output buffer sets (0 = auto)")
    ap.add_argument("--backward", action="store_true",
                    help="time the backward pass (pskv_attn_bwd: dq, dk_suf, dv_suf) instead of the forward pass")
    ap.add_argument("--baseline", default="none", choices=["none", "standard_kv", "lazy_expand"],
                    help="run the paper's comparison layouts through the same kernels instead of the shared prefix: "
                         "standard_kv = prefix K/V physically repeated per candidate and kept resident (Eq. 3); "
                         "lazy_expand = the compact prefix expanded into a per-layer workspace inside every step "
                         "(App. F.5/F.6)")
    ap.add_argument("--preramp", type=int, default=PRERAMP_LAUNCHES,
                    help="untimed launches before the counted warm-up that let the shader clock climb from idle "
                         "(reported as preramp_launches; counter-collection runs set it to 0)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run only a plain element-wise copy of known size (the reference that the "
                         "FETCH_SIZE / WRITE_SIZE counter readings are scaled by)")
    ap.add_argument("--mfma-peak", action="store_true",
                    help="run only the MFMA-only kernel and print the rate the matrix cores sustain on this machine")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on ONE GPU only (the path needs no exchange between "
              "candidates or KV heads, so it would shard by candidates or by KV heads). Use --gpus 1.",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2603_13420_amd import binding as pk, inputs as gen

    pk.load()
    assert torch.cuda.is_available(), "bench.py needs the MI355X"
    if args.copy_calibration:
        # 1 GiB read + 1 GiB written per launch by one element-wise kernel
        n = 1 << 29
        src = torch.zeros(n, dtype=torch.bfloat16, device="cuda:0")
        dst = torch.empty_like(src)
        for _ in range(10):
            torch.mul(src, 1.0, out=dst)
        torch.cuda.synchronize()
        print(json.dumps({"copy_calibration": True, "launches": 10, "read_bytes_per_launch": 2 * n,
                          "written_bytes_per_launch": 2 * n}), flush=True)
        return
    if args.mfma_peak:
        tf = measure_mfma_peak(torch, torch.cuda.current_stream().cuda_stream)
        print(json.dumps({"mfma_only_kernel": True, "measured_tflops": tf, "spec_tflops": PEAK_BF16_TFLOPS,
                          "frac_of_spec": tf / PEAK_BF16_TFLOPS}), flush=True)
        return
    multi = args.workload in gen.MULTI_WORKLOADS
    if args.backward:
        return bench_backward(args)
    if multi:
        w = gen.MULTI_WORKLOADS[args.workload]
        inp = gen.make_multi_inputs(w, pad="zero")
        flops, bytes_, prefix_bytes, exps = alg_counts(w, inp.suf_len, inp.pre_len)
    else:
        w = gen.WORKLOADS[args.workload]
        inp = gen.make_inputs(w, pad="zero", workers=16)
        flops, bytes_, prefix_bytes, exps = alg_counts(w, inp.suf_len)

    # Rotating buffer sets so Q/K/V/O of consecutive calls do not sit in the 256 MB
    # last-level cache: each set is a full copy of the suffix-side tensors and output.
    e = 2 if w.dtype == "bf16" else 4
    set_bytes = (2 * w.B * w.S * w.Hq + 2 * w.B * w.S * w.Hkv) * w.D * e
    nsets = args.sets or int(max(2, min(8, (1 << 30) // max(1, set_bytes) + 1)))
    base = gen.to_device_multi(inp) if multi else gen.to_device(inp)
    sets = []
    for s in range(nsets):
        d = base if s == 0 else {k: (v.clone() if k in ("q", "k_suf", "v_suf") else v) for k, v in base.items()}
        d = dict(d, out=torch.empty_like(base["q"]))
        sets.append(d)
    torch.cuda.synchronize()

    stream = torch.cuda.current_stream().cuda_stream

    # Comparison layouts (single-prefix workloads only, App. F.5 / F.6): every candidate attends to a
    # PRIVATE physical copy of the prefix K/V, which is what the Standard KV cache of Eq. 3 holds; each
    # candidate is then its own "instruction" of the multi-instruction entry point.  standard_kv keeps
    # the B copies resident; lazy_expand makes them inside every step (expand + copy into a workspace
    # that lives for the step only) from the compact cache.  Device memory is READ from torch's
    # allocator, not computed: resident = what the prefix tensors occupy while the steps run,
    # transient = peak during one step above what is allocated between steps.
    mem = {"prefix_kv_bytes_resident": None, "prefix_kv_bytes_transient_per_layer": None}
    if args.baseline != "none":
        assert not multi and w.P > 0, "--baseline applies to the single-prefix workloads"
    if args.baseline == "standard_kv":
        before = torch.cuda.memory_allocated()
        kexp = base["k_pre"][None].expand(w.B, w.P, w.Hkv, w.D).contiguous()
        vexp = base["v_pre"][None].expand(w.B, w.P, w.Hkv, w.D).contiguous()
        torch.cuda.synchronize()
        mem["prefix_kv_bytes_resident"] = torch.cuda.memory_allocated() - before
        for d in sets:
            d["k_pre"], d["v_pre"], d["pre_len"] = kexp, vexp, None
    multi_call = multi or args.baseline == "standard_kv"

    # arguments marshalled once per buffer set: the timed loop is one foreign call per step
    if args.baseline == "lazy_expand":
        prepared = None
    elif multi_call:
        prepared = [pk.PreparedMultiCall(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["pre_len"],
                                         d["suf_len"], d["out"], impl=args.impl, scale=inp.scale, stream=stream)
                    for d in sets]
    else:
        prepared = [pk.PreparedCall(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], d["out"],
                                    impl=args.impl, scale=inp.scale, stream=stream) for d in sets]

    if args.baseline == "lazy_expand":
        def call(i):
            d = sets[i]
            # the per-layer expansion of the compact prefix into a workspace of this step's own ...
            kx = d["k_pre"][None].expand(w.B, w.P, w.Hkv, w.D).contiguous()
            vx = d["v_pre"][None].expand(w.B, w.P, w.Hkv, w.D).contiguous()
            # ... attention over it, and the workspace goes back to the allocator when the step ends
            pk.pskv_attn_fwd_multi(d["q"], d["k_suf"], d["v_suf"], kx, vx, None, d["suf_len"], out=d["out"],
                                   impl=args.impl, scale=inp.scale)
    else:
        def call(i):
            prepared[i]()

    # ---- before anything is timed: one call per buffer set, memory readings, self-check ----
    for i in range(nsets):
        call(i)
    torch.cuda.synchronize()
    if args.baseline == "none":
        mem["prefix_kv_bytes_resident"] = sum(int(base[k].numel()) * e for k in ("k_pre", "v_pre") if base[k] is not None)
        mem["prefix_kv_bytes_transient_per_layer"] = 0
    else:
        if args.baseline == "lazy_expand":
            mem["prefix_kv_bytes_resident"] = sum(int(base[k].numel()) * e for k in ("k_pre", "v_pre"))
        idle = torch.cuda.memory_allocated()
        torch.cuda.reset_peak_memory_stats()
        call(0)
        torch.cuda.synchronize()
        mem["prefix_kv_bytes_transient_per_layer"] = torch.cuda.max_memory_allocated() - idle

    # quick self-check of the timed configuration on a few candidates against the CPU oracle
    from oracle import parity
    if multi:
        which = np.array([0, w.Np - 1])
        sub = inp.take_instructions(which)
        ref = parity.oracle_out_multi(sub)
        cand = (which[:, None] * w.C + np.arange(w.C)[None, :]).reshape(-1)
    else:
        cand = np.array([0, w.B // 2, w.B - 1])
        sub = inp.take(cand)
        ref = parity.oracle_out(sub)
    got = gen.out_to_f64(sets[0]["out"][torch.from_numpy(cand).to("cuda:0")])
    chk = parity.compare(got, ref, sub.suf_len, w.dtype, "bench self-check")

    # what the matrix cores sustain on this machine with nothing else going on
    mfma_measured = (measure_mfma_peak(torch, stream)
                     if w.dtype == "bf16" and args.impl != "simple" and args.preramp > 0 else None)

    # launches timed one at a time, each between its own pair of events (for comparison only)
    isolated_ms = None
    if prepared is not None and not multi_call and args.preramp > 0:
        per_set = []
        for _ in range(max(1, min(20, args.steps // nsets))):
            for i in range(nsets):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                prepared[i]()
                e1.record()
                e1.synchronize()
                per_set.append(e0.elapsed_time(e1))
        isolated_ms = float(np.mean(per_set))

    # ---- clock ramp (untimed, fixed), counted warm-up, timed region ----
    for i in range(args.preramp):
        call(i % nsets)
    for i in range(args.warmup):
        call(i % nsets)
    torch.cuda.synchronize()

    # The timed region: exactly `steps` calls, wall clock bracketed by synchronisation, with
    # HIP events on the launch stream for the kernel-only average.
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ev0.record()
    for i in range(args.steps):
        call(i % nsets)
    ev1.record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ev_ms = ev0.elapsed_time(ev1) / args.steps
    ms_per_step = wall * 1e3 / args.steps

    # Per-launch kernel duration: HIP events over the timed region on the launch stream.  The
    # launches are queued back to back, so the event span divided by the launch count is the
    # average duration of one launch (plus the idle gap between two launches, if any).
    kern_ms = ev_ms

    # The comparison layouts read B private prefix copies: that is their algorithmic traffic
    # (lazy_expand writes them first, too).
    if args.baseline != "none":
        bytes_ += (w.B - 1) * prefix_bytes * (2 if args.baseline == "lazy_expand" else 1)

    cand_per_s = w.B / (ms_per_step * 1e-3)
    if w.dtype == "bf16" and args.impl != "simple":
        compute = {"bound": "mfma", "achieved": flops / (kern_ms * 1e-3) / 1e12, "peak": PEAK_BF16_TFLOPS,
                   "unit": "TFLOP/s"}
    elif w.dtype == "f32":
        compute = {"bound": "alu", "achieved": flops / (kern_ms * 1e-3) / 1e12, "peak": PEAK_F64_TFLOPS,
                   "unit": "TFLOP/s"}
    else:
        compute = {"bound": "alu", "achieved": flops / (kern_ms * 1e-3) / 1e12, "peak": 157.3, "unit": "TFLOP/s"}
    compute["frac"] = compute["achieved"] / compute["peak"]
    compute["alg_flops_per_launch"] = flops
    traffic, mfma_flops, source = offline_counters(HBM_TRAFFIC, w.name, args.impl == "auto" and args.baseline == "none")
    if compute["bound"] == "mfma":
        compute["measured_peak"] = mfma_measured       # the MFMA-only kernel on this machine, this run
        compute["frac_of_measured_peak"] = compute["achieved"] / mfma_measured if mfma_measured else None
        compute["executed_mfma_flops"] = mfma_flops    # SQ_INSTS_VALU_MFMA_MOPS_BF16 * 512 per launch (whole tiles, padding included)
        compute["executed_mfma_flops_source"] = source
    hbm = {"bound": "hbm", "achieved": bytes_ / (kern_ms * 1e-3) / 1e9, "peak": PEAK_HBM_GBS, "unit": "GB/s",
           "alg_bytes_per_launch": bytes_, "prefix_bytes_once": prefix_bytes}
    hbm["frac"] = hbm["achieved"] / hbm["peak"]
    # The binding roofline is the one whose peak gives the longer minimum time for the
    # algorithmic work of this launch; the other one is reported beside it.
    t_compute = flops / (compute["peak"] * 1e12)
    t_hbm = bytes_ / (PEAK_HBM_GBS * 1e9)
    roof, other = (hbm, compute) if t_hbm >= t_compute else (compute, hbm)
    roof["traffic"] = traffic
    roof["traffic_unit"] = "bytes per launch"
    roof["traffic_source"] = source
    roof["kernel_ms"] = kern_ms
    roof["kernel_ms_isolated_launches"] = isolated_ms
    roof["min_ms_at_peak"] = max(t_compute, t_hbm) * 1e3

    line = {
        "metric": "candidate suffixes/sec per attention layer", "value": cand_per_s, "unit": "candidates/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "preramp_launches": args.preramp,
        "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16" if w.dtype == "bf16" and args.impl != "simple" else ("f64" if w.dtype == "f32" else "f32"),
        "data": "synthetic",
        "config": {"workload": w.name, "B": w.B, "P": w.P, "S": w.S, "suffix_len": [w.len_lo, w.len_hi],
                   "Hq": w.Hq, "Hkv": w.Hkv, "D": w.D, "impl": args.impl, "buffer_sets": nsets,
                   "seed": w.seed, "prefix_layout": args.baseline if args.baseline != "none" else "shared (PSKV)",
                   **mem, "memory_source": "torch.cuda.memory_allocated / max_memory_allocated around one step",
                   **({"instructions": w.Np, "candidates_per_instruction": w.C,
                                       "prefix_len": [w.pre_lo, w.pre_hi]} if multi else {})},
        "achieved_tflops": flops / (ms_per_step * 1e-3) / 1e12,
        "event_ms_per_step": ev_ms,
        "roofline": roof, "roofline_" + other["bound"]: other,
        "exp_per_launch": exps,
        "self_check": chk,
    }
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline_multi(inp) if multi else cpu_baseline(inp)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
