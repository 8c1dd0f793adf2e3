#!/usr/bin/env python3
"""Benchmark of the denoising hot path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload cfg4|cfg2|cfg3a|cfg5a]

A step is one fc_denoise_step over one batch of synthetic input (text projection,
timestep conditioning, patch embedding, every transformer block, output head,
guidance and DDIM update), inputs resident in HBM.  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0      # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0


def ln_bytes_per_element(launches: int, esz: int) -> int:
    """Bytes per residual-stream element that the LayerNorm launches of one step move: every
    launch reads x (fp32) and writes its output (activation type); it also reads the branch
    outputs not yet added to x, one after a launch that wrote x back (or the first), two
    otherwise, and writes x back (fp32) when it has read two.  The last launch never writes x."""
    total, pending = 0, 0
    for i in range(launches):
        total += 4 + esz + pending * esz
        if pending == 2 and i < launches - 1:
            total += 4
        if pending == 2:
            pending = 0
        pending += 1
    return total


def measured_traffic(kernel):
    """(HBM bytes per launch of `kernel`, where the figure comes from): the bytes are replayed
    from the committed rocprofv3 counter summary, not counted in this run; (None, reason) when
    there is no summary or the kernel source has changed since the counters were taken."""
    import glob
    import hashlib
    for path in sorted(glob.glob(os.path.join(ROOT, "profiles", "*hbm_traffic.txt"))):
        kv = {}
        for line in open(path):
            if "=" in line and not line.startswith("#"):
                k, v = line.split("=", 1)
                kv[k.strip()] = v.strip()
        if f"{kernel}.fetch_bytes" not in kv:
            continue
        src = os.path.join(ROOT, "paper_2501_04012_amd", "csrc", "attention.hip")
        rel = os.path.relpath(path, ROOT)
        if hashlib.sha256(open(src, "rb").read()).hexdigest() != kv.get(f"{kernel}.source_sha256"):
            return None, f"{rel}: stale (the kernel source changed after the counters were taken)"
        return (float(kv[f"{kernel}.fetch_bytes"]) + float(kv[f"{kernel}.write_bytes"]),
                f"replayed from {rel} (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE, taken {kv.get('date', 'date not recorded')}); "
                f"not counted in this run")
    return None, "no counter summary under profiles/"


def cpu_baseline(w, weights, lat, cond):
    """The oracle (fp32 arithmetic) on the host cores, on a bounded sample of the same
    workload, converted to steps/s."""
    from oracle import dit, sampler
    from paper_2501_04012_amd import synth
    try:
        from threadpoolctl import threadpool_info
        cores = max([p.get("num_threads", 1) for p in threadpool_info()] or [os.cpu_count() or 1])
    except Exception:
        cores = os.cpu_count() or 1
    cfg = w.model
    W32 = {k: np.asarray(v, dtype=np.float32) for k, v in weights.items()}
    if cfg.attn_mode == synth.ATTN_FULL3D_CONCAT and cfg.depth == 1:
        # the whole block, every row: one forward of the workload's one sample is the whole step
        # (about half a minute on 16 host threads; the update itself is negligible)
        t0 = time.perf_counter()
        dit.forward(cfg, W32, lat[0].astype(np.float32), cond[0].astype(np.float32), 500, dtype=None)
        step_s = time.perf_counter() - t0
        sample = (f"fp32 oracle forward of the whole block, all {cfg.video_tokens} rows, once ({step_s:.1f}s): "
                  f"one step of the workload, nothing extrapolated")
    else:
        # one forward of one sample (through at most 28 blocks: about 10 s at the 1152-wide
        # shapes), scaled to depth and batch
        from dataclasses import replace
        d = min(cfg.depth, 28)
        cfg_s = replace(cfg, depth=d)
        Ws = {k: v for k, v in W32.items() if not k.startswith("blk") or int(k[3:k.index(".")]) < d}
        t0 = time.perf_counter(); dit.forward(cfg_s, Ws, lat[0].astype(np.float32), cond[0].astype(np.float32), 500,
                                              dtype=None)
        t1 = time.perf_counter()
        forwards = lat.shape[0] * (2 if w.null_seed is not None else 1)
        step_s = (t1 - t0) * (cfg.depth / d) * forwards
        sample = (f"fp32 oracle forward of one sample through {d} of {cfg.depth} blocks ({t1 - t0:.1f}s), "
                  f"scaled by depth and by {forwards} forwards per step")
    cpu_model = ""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.lower().startswith("model name"):
                    cpu_model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"value": 1.0 / step_s, "unit": "steps/s", "cores": int(cores), "kind": "oracle", "sample": sample,
            "host_cpus": os.cpu_count() or 0, "cpu_model": cpu_model}


def resume_cfg5a(k=10):
    """One fc_denoise_resume call of the cfg5a workload (4 requests x guidance pair, 28 blocks of
    the 1152-wide factorized model, 50-step schedule) from step k, wall clock."""
    import torch
    import paper_2501_04012_amd as fc
    from paper_2501_04012_amd import synth
    w = synth.WORKLOADS["cfg5a"]
    cfg = w.model
    weights = synth.make_weights(cfg, w.weight_seed)
    lat, cond, null = synth.workload_inputs(w)
    den = fc.Denoiser(cfg, weights, lat.shape[0], True)
    del weights
    d_cond, d_null = torch.from_numpy(cond).cuda(), torch.from_numpy(null).cuda()
    d_lat0 = torch.from_numpy(lat).cuda()
    d_lat = d_lat0.clone()
    den.resume(d_lat, d_cond, d_null, w.schedule, w.schedule.num_steps - 2)       # warm-up: two steps
    d_lat.copy_(d_lat0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    den.resume(d_lat, d_cond, d_null, w.schedule, k)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3
    n = w.schedule.num_steps - k
    forwards = lat.shape[0] * 2
    tflops = synth.forward_flops(cfg)["total"] * forwards * n / (ms * 1e-3) / 1e12
    den.close()
    return {"k": k, "steps": n, "requests": int(lat.shape[0]), "ms": ms, "ms_per_step": ms / n, "tflops": tflops,
            "pct_peak": 100.0 * tflops / PEAK_BF16_TFLOPS}


def cache_restore_bench(args):
    """Secondary measurement (--cache-restore): the entry points that produce the `latent`
    argument of a resume, at the paper's latent shape (64 x 40 x 64 x 4, Sec. 2.3) and on a
    batch of 256 such latents, where the HBM rate shows.  One JSON line."""
    import torch
    import paper_2501_04012_amd as fc
    torch.cuda.set_device(0)
    T, H, W, C = 64, 40, 64, 4
    F = H * W * C
    out = {}
    for label, R in (("one_latent", 1), ("batch_256", 256)):
        frames = R * T
        g = torch.Generator(device="cuda").manual_seed(1)
        xo = torch.randn(frames, H, W, C, device="cuda", generator=g)
        xb = torch.randn(frames, H, W, C, device="cuda", generator=g)
        # masks shaped like a segmented object: a rectangle per frame that drifts with the frame
        # index; the background mask is its complement grown by one pixel (a slight misalignment)
        obj = np.zeros((frames, H, W), dtype=bool)
        bgm = np.ones((frames, H, W), dtype=bool)
        for f in range(frames):
            x0 = 8 + (f % T) // 4
            obj[f, 10:30, x0:x0 + 24] = True
            bgm[f, 9:31, x0 - 1:x0 + 25] = False
        mo = torch.from_numpy(np.packbits(obj.reshape(-1), bitorder="little")).cuda()
        mb = torch.from_numpy(np.packbits(bgm.reshape(-1), bitorder="little")).cuda()
        dst = torch.empty_like(xo)

        def timed(fn, reps=args.steps):
            for _ in range(args.warmup):
                fn()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(reps):
                fn()
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / reps

        ms = timed(lambda: fc.fc_cache_stitch(xo, xb, mo, mb, dst, frames * H * W, C))
        nbytes = frames * F * 4 * 2 + 2 * mo.numel()           # one source read and one write per element, both masks
        res = {"stitch": {"ms": ms, "gbps": nbytes / ms / 1e6}}
        if R == 1:
            n_base, n_extra = 8, 4
            src = [0] + [1 + (t % n_base) if t % 5 else -(1 + t % n_extra) for t in range(1, T)]
            ms = timed(lambda: fc.fc_cache_decompress(xo[0], xb[:n_base], n_base, 0.75, xb[8:8 + n_extra], n_extra, src,
                                                      T, F, dst))
            reads = sum(2 if c > 0 else 1 for c in src)
            res["decompress"] = {"ms": ms, "gbps": (reads + T) * F * 4 / ms / 1e6}
            ws = torch.empty(fc.fc_cache_workspace_bytes(T), dtype=torch.uint8, device="cuda")
            a = torch.zeros(1, device="cuda")
            ms = timed(lambda: fc.fc_cache_alpha(xo[0], xo[1:1 + n_base], xb[:n_base], n_base, F, a, ws))
            res["alpha"] = {"ms": ms, "gbps": (2 * n_base + 1) * F * 4 / ms / 1e6}
            sim = torch.empty(T, T, device="cuda")
            ms = timed(lambda: fc.fc_cache_frame_similarity(xo, T, F, sim, ws))
            res["frame_similarity"] = {"ms": ms, "gbps": T * F * 4 / ms / 1e6}
        out[label] = res
    best = out["batch_256"]["stitch"]["gbps"]
    print(json.dumps({
        "metric": "cache restore (stitch) GB/s on 256 paper-shaped latents", "value": best, "unit": "GB/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": out["batch_256"]["stitch"]["ms"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "cache_restore", "latent": [T, H, W, C]},
        "roofline": {"kernel": "k_stitch", "bound": "hbm", "achieved": best, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                     "frac": best / PEAK_HBM_GBS, "traffic": None},
        "ops": out}))


def hbm_ops_bench(args):
    """Secondary measurement (--hbm-ops): the two HBM-bound operators of a step whose real
    shapes are too small to show a rate, LayerNorm+modulate and the guidance + DDIM update,
    timed at the real shape (latency) and on a scaled batch (GB/s).  One JSON line."""
    import torch
    import paper_2501_04012_amd as fc
    torch.cuda.set_device(0)

    def timed(fn, reps=args.steps):
        for _ in range(args.warmup):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    out = {}
    g = torch.Generator(device="cuda").manual_seed(1)
    # guidance + DDIM update: per element read x, eps_c, eps_u and write x = 16 bytes
    coef = fc.fc_schedule_coefficients(fc.synth.Schedule(), 25)[0]
    for label, n in (("cfg_ddim real (cfg5a: 4 x 16x32x32x4)", 4 * 65536), ("cfg_ddim real (cfg4 latent)", 13 * 60 * 90 * 16),
                     ("cfg_ddim scaled (512 latents of 16x32x32x4)", 512 * 65536)):
        x = torch.randn(n, device="cuda", generator=g)
        ec = torch.randn(n, device="cuda", generator=g)
        eu = torch.randn(n, device="cuda", generator=g)
        ms = timed(lambda: fc.fc_op_cfg_ddim(x, ec, eu, None, n, 7.5, coef))
        out[label] = {"ms": ms, "gbps": 16.0 * n / ms / 1e6}
    # LayerNorm+modulate with the pending residual add: per element read x (4), read y (2),
    # write x (4), write out (2) = 12 bytes; without the add: read x, write out = 6 bytes
    for label, M, D in (("ln_modulate real (cfg4: 17776 x 3072)", 17776, 3072),
                        ("ln_modulate scaled (cfg4 rows x 8)", 8 * 17776, 3072),
                        ("ln_modulate real (cfg5a: 32768 x 1152)", 32768, 1152),
                        ("ln_modulate scaled (cfg5a rows x 16)", 16 * 32768, 1152)):
        x = torch.randn(M, D, device="cuda", generator=g)
        y = (0.01 * torch.randn(M, D, device="cuda", generator=g)).to(torch.bfloat16)
        sh = torch.randn(D, device="cuda", generator=g)
        sc = torch.randn(D, device="cuda", generator=g)
        o = torch.empty(M, D, device="cuda", dtype=torch.bfloat16)
        ms = timed(lambda: fc.fc_op_layernorm_modulate(fc.FC_BF16, x, None, sh, sc, o, M, D, 1e-6))
        ms_add = timed(lambda: fc.fc_op_layernorm_modulate(fc.FC_BF16, x, y, sh, sc, o, M, D, 1e-6))
        out[label] = {"ms": ms, "gbps": 6.0 * M * D / ms / 1e6, "with_residual_add": {"ms": ms_add, "gbps": 12.0 * M * D / ms_add / 1e6}}
    best = out["ln_modulate scaled (cfg4 rows x 8)"]["with_residual_add"]
    print(json.dumps({
        "metric": "LayerNorm+modulate (with residual add) GB/s on a scaled batch", "value": best["gbps"], "unit": "GB/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": best["ms"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": "hbm_ops"},
        "roofline": {"kernel": "k_ln_modulate", "bound": "hbm", "achieved": best["gbps"], "peak": PEAK_HBM_GBS,
                     "unit": "GB/s", "frac": best["gbps"] / PEAK_HBM_GBS, "traffic": None},
        "ops": out}))


def mfma_ceiling_bench(args):
    """Secondary measurement (--mfma-ceiling): what the part at hand sustains.
    (1) The library's pipe-rate microbenchmark: independent bf16 MFMA chains, of 32x32x16 (the
    attention kernels) and of 16x16x32 (the products), on random and on constant operands, v_exp_f32 streams, both in one wave, and MFMA waves beside
    exponential waves on the same SIMDs, each with the shader clock it ran at.
    (2) Yardsticks, not on the product path: torch.matmul (bf16, the vendor's GEMM library) on
    the four GEMM shapes of the full-3D configuration and torch's fused attention on its
    attention shape, timed on the same box.  One JSON line."""
    import torch
    import paper_2501_04012_amd as fc
    torch.cuda.set_device(0)
    g = torch.Generator(device="cuda").manual_seed(1)

    def timed(fn, reps):
        for _ in range(2):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    rnd = torch.randn(4096, device="cuda", generator=g).to(torch.bfloat16)
    const = torch.ones(4096, device="cuda", dtype=torch.bfloat16)
    iters = 200000
    pipes = {}
    for label, ops, ma, mb, blocks in (
            ("mfma_random_operands_2_waves_per_simd", rnd, 1, 1, 256),
            ("mfma_16x16x32_random_operands_2_waves_per_simd", rnd, 4, 4, 256),
            ("mfma_random_operands_4_waves_per_simd", rnd, 1, 1, 512),
            ("mfma_constant_operands_2_waves_per_simd", const, 1, 1, 256),
            ("mfma_16x16x32_constant_operands_2_waves_per_simd", const, 4, 4, 256),
            ("exp_only_2_waves_per_simd", rnd, 2, 2, 256),
            ("mfma_and_exp_in_one_wave", rnd, 3, 3, 256),
            ("mfma_waves_beside_exp_waves", rnd, 1, 2, 256)):
        sink = torch.empty(blocks * 512, device="cuda")
        clocks = torch.zeros(blocks * 16, dtype=torch.int64, device="cuda")
        ms = timed(lambda: fc.fc_bench_pipe_rates(ops, iters, ma, mb, blocks, sink, clocks), 3)
        c = clocks.cpu().numpy().reshape(-1, 2).astype(np.float64)
        mfma_waves = blocks * (4 * (ma in (1, 3, 4)) + 4 * (mb in (1, 3, 4)))
        exp_waves = blocks * (4 * (ma in (2, 3)) + 4 * (mb in (2, 3)))
        r = {"ms": ms, "shader_clock_ghz": float(np.median(c[:, 0] / np.maximum(c[:, 1], 1.0)) * 0.1)}
        if mfma_waves:
            r["mfma_tflops"] = mfma_waves * iters * 4 * 32768.0 / (ms * 1e-3) / 1e12
        if exp_waves:
            r["exp_per_ns"] = exp_waves * iters * 8 * 64.0 / (ms * 1e6)
        if ma != mb:        # the two halves finish at different times: per-half durations from the wave clocks
            half = c.reshape(blocks, 8, 2)
            r["first_half_ms"] = float(np.median(half[:, :4, 1])) * 1e-5
            r["second_half_ms"] = float(np.median(half[:, 4:, 1])) * 1e-5
        pipes[label] = r

    yard = {}
    M = 17776
    for name, K, N in (("qkv", 3072, 9216), ("proj", 3072, 3072), ("fc1", 3072, 12288), ("fc2", 12288, 3072)):
        a = (torch.randn(M, K, device="cuda", generator=g)).to(torch.bfloat16)
        wt = (0.02 * torch.randn(N, K, device="cuda", generator=g)).to(torch.bfloat16)
        o = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
        ms = timed(lambda: torch.matmul(a, wt.t(), out=o), 10)
        yard["torch_matmul_" + name] = {"m_n_k": [M, N, K], "ms": ms, "tflops": 2.0 * M * N * K / (ms * 1e-3) / 1e12}
        # the library's own linear on the same operands, same timing loop
        ms = timed(lambda: fc.fc_op_linear(fc.FC_BF16, a, wt, None, None, o, M, N, K, 0), 10)
        yard["fc_op_linear_" + name] = {"m_n_k": [M, N, K], "ms": ms, "tflops": 2.0 * M * N * K / (ms * 1e-3) / 1e12}
        del a, wt, o
    try:
        H, Nt, d = 48, 17776, 64
        q = torch.randn(1, H, Nt, d, device="cuda", generator=g).to(torch.bfloat16)
        k = torch.randn(1, H, Nt, d, device="cuda", generator=g).to(torch.bfloat16)
        v = torch.randn(1, H, Nt, d, device="cuda", generator=g).to(torch.bfloat16)
        ms = timed(lambda: torch.nn.functional.scaled_dot_product_attention(q, k, v), 3)
        yard["torch_sdpa_full3d"] = {"heads_tokens_d": [H, Nt, d], "ms": ms, "tflops": 4.0 * H * Nt * Nt * d / (ms * 1e-3) / 1e12}
        o = torch.empty(H, Nt, d, device="cuda", dtype=torch.bfloat16)
        ms = timed(lambda: fc.fc_op_attention(fc.FC_BF16, q[0], k[0], v[0], o, H, Nt, Nt, d, 0), 3)
        yard["fc_op_attention_full3d"] = {"heads_tokens_d": [H, Nt, d], "ms": ms,
                                          "tflops": 4.0 * H * Nt * Nt * d / (ms * 1e-3) / 1e12}
    except Exception as exc:                      # the yardstick is optional: some builds carry no fused attention
        yard["torch_sdpa_full3d"] = {"error": repr(exc)[:200]}
    best = pipes["mfma_random_operands_2_waves_per_simd"]
    print(json.dumps({
        "metric": "sustained bf16 MFMA TFLOP/s of independent 32x32x16 chains on random operands", "value": best["mfma_tflops"],
        "unit": "TFLOP/s", "n_gpus": 1, "steps": 3, "warmup": 2, "ms_per_step": best["ms"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": "mfma_ceiling"},
        "roofline": {"kernel": "k_pipe_rates", "bound": "mfma", "achieved": best["mfma_tflops"], "peak": PEAK_BF16_TFLOPS,
                     "unit": "TFLOP/s", "frac": best["mfma_tflops"] / PEAK_BF16_TFLOPS, "traffic": None},
        "pipes": pipes, "yardsticks": yard}))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="cfg4")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-resume", action="store_true",
                    help="skip the whole cfg5a resume call that the default (cfg4) line also reports")
    ap.add_argument("--cache-restore", action="store_true",
                    help="time the cache-restore entry points instead of a denoising workload")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="also run one plain device copy of this size (a known-size kernel for scaling HBM counters)")
    ap.add_argument("--mfma-ceiling", action="store_true",
                    help="microbenchmarks of the matrix / vector pipes and vendor-library yardsticks instead")
    ap.add_argument("--hbm-ops", action="store_true",
                    help="time LayerNorm+modulate and the guidance+DDIM update at real and scaled shapes instead")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: the library runs on one GPU only (no sharding, no collectives); use --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2501_04012_amd as fc
    from paper_2501_04012_amd import synth

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    if args.cache_restore:
        cache_restore_bench(args)
        return
    if args.hbm_ops:
        hbm_ops_bench(args)
        return
    if args.mfma_ceiling:
        mfma_ceiling_bench(args)
        return
    torch.cuda.set_device(0)
    w = synth.WORKLOADS[args.workload]
    cfg = w.model
    weights = synth.make_weights(cfg, w.weight_seed)
    lat, cond, null = synth.workload_inputs(w)
    R = lat.shape[0]
    use_cfg = null is not None
    den = fc.Denoiser(cfg, weights, R, use_cfg)
    d_lat0 = torch.from_numpy(lat).cuda()
    d_cond = torch.from_numpy(cond).cuda()
    d_null = torch.from_numpy(null).cuda() if use_cfg else None
    d_lat = d_lat0.clone()

    if args.copy_calibration_mib:
        src = torch.empty(args.copy_calibration_mib << 20, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    for _ in range(args.warmup):
        d_lat.copy_(d_lat0)
        den.step(d_lat, d_cond, d_null, w.schedule, w.step)
    torch.cuda.synchronize()

    # untimed pass with every launch group bracketed: the per-kernel breakdown, and which
    # kernel dominates
    psteps = max(1, min(args.steps, 3))
    fc.fc_profile_select(den.model, None)
    fc.fc_profile_enable(den.model, True)
    d_lat.copy_(d_lat0)
    for _ in range(psteps):
        den.step(d_lat, d_cond, d_null, w.schedule, w.step)
    torch.cuda.synchronize()
    prof = fc.fc_profile_read(den.model)
    kernels = {}
    for name, (ms, cnt) in prof.items():
        if cnt:
            kernels[name] = {"ms_per_step": ms / psteps, "avg_launch_ms": ms / cnt, "launches_per_step": cnt / psteps}
    dom = max(kernels, key=lambda k: kernels[k]["ms_per_step"])

    # timed region: exactly K steps; only the dominant kernel is bracketed by HIP events
    # (on the stream it is launched on), so the wall clock carries two event records per
    # launch of that kernel and nothing else
    fc.fc_profile_select(den.model, dom)
    d_lat.copy_(d_lat0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        den.step(d_lat, d_cond, d_null, w.schedule, w.step)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    dom_ms, dom_cnt = fc.fc_profile_read(den.model)[dom]
    fc.fc_profile_enable(den.model, False)
    fc.fc_profile_select(den.model, None)
    dom_launch_ms = dom_ms / dom_cnt

    # per-step spread (after the timed region, no kernel bracketed): one event pair per step
    # on the stream the steps run on; median and minimum over min(K, 20) steps
    d_lat.copy_(d_lat0)
    pairs = []
    for _ in range(max(1, min(args.steps, 20))):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        den.step(d_lat, d_cond, d_null, w.schedule, w.step)
        e1.record()
        pairs.append((e0, e1))
    torch.cuda.synchronize()
    per_step = sorted(a.elapsed_time(b) for a, b in pairs)

    # workloads that are a cache-hit resume: the whole loop from each of their k, one call each
    # (text projection and cross-attention keys/values once per call, then N - k steps)
    resume = {}
    for k in getattr(w, "resume_k", ()) or ():
        d_lat.copy_(d_lat0)
        torch.cuda.synchronize()
        r0 = time.perf_counter()
        den.resume(d_lat, d_cond, d_null, w.schedule, k)
        torch.cuda.synchronize()
        r1 = time.perf_counter()
        n = w.schedule.num_steps - k
        resume["k=%d" % k] = {"steps": n, "ms": (r1 - r0) * 1e3, "ms_per_step": (r1 - r0) * 1e3 / n}

    ms_per_step = (t1 - t0) * 1e3 / args.steps
    forwards = R * (2 if use_cfg else 1)
    fl = synth.forward_flops(cfg)
    step_flops = fl["total"] * forwards
    tflops = step_flops / (ms_per_step * 1e-3) / 1e12

    per_launch_flops = {
        "attn_full3d": fl["block_attention"] * forwards,
        "attn_spatial": 4.0 * cfg.video_tokens * cfg.spatial_tokens * cfg.hidden * forwards,
        "attn_cross": 4.0 * cfg.video_tokens * cfg.text_len * cfg.hidden * forwards,
        "gemm_qkv": 2.0 * cfg.seq_tokens * cfg.hidden * 3 * cfg.hidden * forwards,
        "gemm_fc1": 2.0 * cfg.seq_tokens * cfg.hidden * cfg.mlp_dim * forwards,
        "gemm_fc2": 2.0 * cfg.seq_tokens * cfg.hidden * cfg.mlp_dim * forwards,
        "gemm_proj": 2.0 * cfg.seq_tokens * cfg.hidden * cfg.hidden * forwards,
    }
    for k, f in per_launch_flops.items():
        if k in kernels:
            kernels[k]["tflops"] = f / (kernels[k]["avg_launch_ms"] * 1e-3) / 1e12
    # HBM-bound launch groups: algorithmic bytes per step (what has to cross HBM once) over their time
    esz = 2 if cfg.dtype == synth.DT_BF16 else 4
    elems = forwards * cfg.seq_tokens * cfg.hidden
    factorized = cfg.attn_mode == synth.ATTN_FACTORIZED_CROSS
    ln_launches = (4 if factorized else 2) * cfg.depth + 1
    nmod = 9 if factorized else 6
    lat_elems = R * cfg.frames * cfg.height * cfg.width * cfg.channels
    per_step_bytes = {
        "ln_modulate": elems * ln_bytes_per_element(ln_launches, esz),
        "patch_embed": forwards * cfg.video_tokens * cfg.hidden * 4,
        "timestep_modulation": (cfg.depth * nmod + 2) * cfg.hidden * cfg.hidden * esz
                               + (cfg.t_embed_dim + cfg.hidden) * cfg.hidden * esz,
        "cfg_ddim": lat_elems * (16 if use_cfg else 12),
        "attn_temporal": cfg.depth * 4 * forwards * cfg.video_tokens * cfg.hidden * esz,
        "attn_cross": cfg.depth * 2 * forwards * cfg.video_tokens * cfg.hidden * esz,
    }
    for k, nbytes in per_step_bytes.items():
        if k in kernels:
            kernels[k]["gbps"] = nbytes / (kernels[k]["ms_per_step"] * 1e-3) / 1e9
    if dom in per_launch_flops:
        ach = per_launch_flops[dom] / (dom_launch_ms * 1e-3) / 1e12
        traffic, traffic_source = measured_traffic(dom)
        roofline = {"kernel": dom, "bound": "mfma", "achieved": ach, "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                    "frac": ach / PEAK_BF16_TFLOPS, "traffic": traffic, "traffic_source": traffic_source,
                    "avg_launch_ms": dom_launch_ms, "launches": int(dom_cnt)}
    else:
        roofline = {"kernel": dom, "bound": "hbm", "achieved": None, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                    "frac": None, "traffic": None}

    out = {
        "metric": "denoising steps/s per video + attention/GEMM TFLOP/s (% of MI355X bf16 peak)",
        "value": 1e3 / ms_per_step, "unit": "steps/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16" if cfg.dtype == synth.DT_BF16 else "f32", "data": "synthetic",
        "config": {"workload": args.workload, "requests": R, "guidance_pair": use_cfg,
                   "tokens": cfg.seq_tokens, "hidden": cfg.hidden, "heads": cfg.heads, "depth": cfg.depth,
                   "attn_mode": "full3d_concat" if cfg.attn_mode else "factorized_cross"},
        "ms_per_step_median": per_step[len(per_step) // 2], "ms_per_step_min": per_step[0],
        "video_steps_per_s": R * 1e3 / ms_per_step,
        "tflops": tflops, "pct_bf16_peak": 100.0 * tflops / PEAK_BF16_TFLOPS,
        "step_tflop": step_flops / 1e12,
        "roofline": roofline,
        "kernels": kernels,
    }
    if resume:
        out["resume"] = resume
    den.close()
    if args.workload == "cfg4" and not args.no_resume:
        # the computation the cache resumes, beside the headline block: one whole
        # fc_denoise_resume of the 28-block stack from k = 10 (4 requests x guidance pair)
        del den, d_lat, d_lat0, d_cond
        torch.cuda.empty_cache()
        out["resume_cfg5a"] = resume_cfg5a()
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w, weights, lat, cond)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
