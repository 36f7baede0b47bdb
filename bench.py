#!/usr/bin/env python3
"""Throughput of Bluebild standard synthesis on one MI355X.

Workload (default): the LOFAR-like single-channel configuration -- 512
stations over 50 km, 100 epochs over 6 h of Earth rotation, 1024 x 1024
pixels over 10 degrees, all 512 eigenpairs in 8 positive + 1 negative
k-means levels, complex64 contraction with FP64 phase arguments.  Inputs are
synthetic (seeded sims), built on the host; the eigenpairs come from the
library's own FP64 GPU pre-step before the timed region.

A step is one pass of the synthesis hot path over the whole job (staging of
every epoch plus one batched synthesis launch over all 100 epochs), with all
inputs resident in HBM.  Prints one JSON line on stdout; progress goes to
stderr.

    python bench.py [--steps K] [--warmup W] [--precision fp32|bf16x3]
"""

import argparse
import json
import os
import sys
import time

import numpy as np

FP32_PEAK_TFLOPS = 157.3      # MI355X dense FP32 matrix
F16_PEAK_TFLOPS = 2516.6      # MI355X dense 16-bit matrix (fp16 and bf16)

ROOT = os.path.dirname(os.path.abspath(__file__))
KERNEL_SOURCE = os.path.join(ROOT, "paper_2310_09200_amd", "csrc", "synth_kernels.hip")
# Counter summary of the synthesis kernel on this workload (rocprofv3 --pmc
# FETCH_SIZE / WRITE_SIZE, calibrated by a device copy of known size; MFMA busy;
# transcendental instructions).  It names the sha256 of the kernel code the
# counters were taken on (the source without its // comments and blank lines,
# so that a comment edit keeps the figures and any code edit drops them); its
# figures are used only while that code is the current one, and reported as
# null otherwise.
COUNTER_SUMMARY = os.path.join(ROOT, "profiles", "synth_fwd_c2_counters.md")


def kernel_code_sha256(path=KERNEL_SOURCE):
    import hashlib
    code = []
    with open(path) as f:
        for ln in f.read().splitlines():
            i = ln.find("//")
            if i >= 0:
                ln = ln[:i]
            ln = ln.rstrip()
            if ln.strip():
                code.append(ln)
    return hashlib.sha256("\n".join(code).encode()).hexdigest()


def counter_figures(mode):
    """{name: value} for ``mode`` from the counter summary, or None when it is absent or stale.

    The summary carries lines ``kernel_code_sha256: <hex>`` and
    ``<mode>.<name>: <value>`` (bytes per launch, MFMA busy fraction,
    transcendental wave instructions per launch, ...).
    """
    try:
        with open(COUNTER_SUMMARY) as f:
            lines = f.read().splitlines()
    except OSError:
        return None
    sha, out = None, {}
    for ln in lines:
        ln = ln.strip().strip("`")
        if ln.startswith("kernel_code_sha256:"):
            sha = ln.split(":", 1)[1].strip()
        elif ln.startswith(mode + ".") and ":" in ln:
            k, v = ln[len(mode) + 1:].split(":", 1)
            try:
                out[k.strip()] = float(v)
            except ValueError:
                pass
    if sha is None or sha != kernel_code_sha256() or not out:
        return None
    return out


def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def gpu_eigenpairs(torch, ctx, w, insts, n_eig, n_pos_levels):
    """Eigenpairs of every instance from the library's FP64 GPU pre-step (untimed set-up).

    Level intervals: exact k-means of the first epoch's eigenvalues (plus one
    level for the non-positive ones), used for every epoch.  Returns
    (intervals, items for Batch, pre-step milliseconds per epoch).
    """
    from paper_2310_09200_amd import StandardSynthesis
    from sims.levels import kmeans1d_intervals
    L = insts[0].x.shape[0]
    probe = StandardSynthesis(ctx, w.pix[:1], 1, 1, L, n_eig)
    _, lam0, _, _ = probe.prestep(insts[0].x, insts[0].wl, insts[0].V, n_eig, np.array([[-np.inf, np.inf]]))
    intervals = kmeans1d_intervals(lam0.cpu().numpy(), n_pos_levels, negative_level=True)
    probe.close()
    pre = StandardSynthesis(ctx, w.pix[:1], intervals.shape[0], 1, L, n_eig)
    # one library call per epoch (each waits for its own eigensolver status), on a few epochs
    n_single = min(4, len(insts))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for inst in insts[:n_single]:
        pre.prestep(inst.x, inst.wl, inst.V, n_eig, intervals)
    torch.cuda.synchronize()
    single_ms = (time.perf_counter() - t0) * 1e3 / n_single
    # every epoch in one call: one strided-batched eigensolve, one wait (inputs uploaded beforehand)
    xs = torch.as_tensor(np.stack([inst.x for inst in insts])).to(ctx.device)
    Vs = torch.as_tensor(np.stack([inst.V for inst in insts])).to(ctx.device)
    wls = [inst.wl for inst in insts]
    pre.prestep_batched(xs[:2], wls[:2], Vs[:2], n_eig, intervals)   # warm-up
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    W, lam, d, lev = pre.prestep_batched(xs, wls, Vs, n_eig, intervals)
    torch.cuda.synchronize()
    batched_ms = (time.perf_counter() - t0) * 1e3 / len(insts)
    items = [(0, inst.x, inst.wl, W[i], d[i], lev[i]) for i, inst in enumerate(insts)]
    pre.close()
    del xs, Vs
    return intervals, items, {"batched_ms_per_epoch": batched_ms, "single_call_ms_per_epoch": single_ms,
                              "epochs": len(insts), "single_call_epochs": n_single}


def build_inputs(args, torch, dev):
    from paper_2310_09200_amd import Context
    from sims import configs

    w = configs.c2(n_steps=args.epochs, n_side=args.n_side)
    ctx = Context(0)
    t0 = time.time()
    insts = [w.instance(i) for i in range(args.epochs)]
    log(f"simulated {len(insts)} visibility matrices in {time.time() - t0:.1f}s")
    intervals, items, pre = gpu_eigenpairs(torch, ctx, w, insts, 512, 8)
    log(f"GPU FP64 pre-step (Gram + zhegvd + selection): {pre['batched_ms_per_epoch']:.2f} ms per epoch batched "
        f"over {pre['epochs']} epochs, {pre['single_call_ms_per_epoch']:.1f} ms in one call per epoch")
    return ctx, w, intervals, items, insts, pre


def measure_phase_peak(torch, ctx, w, items, reps=4, steps=3):
    """Peak phase-generation rate of this device: the probe kernel evaluates every (antenna, pixel) phase of
    the workload's first epoch with the synthesis kernel's arithmetic and no contraction beside it.
    Returns (pairs per second, ms per probe call, pairs per call)."""
    from paper_2310_09200_amd import phase_probe
    _, x, wl = items[0][:3]
    pix = torch.as_tensor(w.pix).to(ctx.device)  # the per-call column-major copy stays on the device
    out = phase_probe(ctx, x, wl, pix, reps)  # warm-up
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        phase_probe(ctx, x, wl, pix, reps, out)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    pairs = float(x.shape[0]) * w.n_pix * reps
    return pairs / (ms / 1000.0), ms, pairs


def time_modes(args, torch, ctx, w, items, modes, n_levels, sel, steps=None, warmup=None):
    """Time every contraction mode, interleaved step by step (same thermal / power state for all).

    After the timed steps each handle is reset and runs the timed launch once
    more; its images at the sample pixels ``sel`` are what the oracle check
    compares.  Returns {mode: (ms per step, synthesis kernel ms, staging ms,
    products per pixel, sampled images (n_levels, len(sel)))}.
    """
    from paper_2310_09200_amd import Batch, StandardSynthesis
    steps = args.steps if steps is None else steps
    warmup = args.warmup if warmup is None else warmup
    batch = Batch(items, ctx.device)
    L = max(int(i.n_ant) for i in batch.inst)
    K = max(int(i.n_eig) for i in batch.inst)
    handles = {m: StandardSynthesis(ctx, w.pix, n_levels, 1, L, K, m) for m in modes}
    tune = {}
    if not args.no_autotune:
        # tile shapes timed on a few of the epochs (each epoch is the same work shape), fastest kept
        sub = Batch(items[:min(8, len(items))], ctx.device)
        for m in modes:
            t0 = time.perf_counter()
            table = handles[m].autotune_batched(sub, reps=1)
            tune[m] = {"tiles": handles[m].tiles, "ms_per_launch_by_class_and_tile": table,
                       "epochs_timed": len(sub.inst), "seconds": time.perf_counter() - t0}
            log(f"{m}: autotuned tiles {handles[m].tiles} from {table}")
    for _ in range(warmup):
        for m in modes:
            handles[m].collect_eig_batched(batch)
    torch.cuda.synchronize()
    wall = {m: [] for m in modes}
    kern = {m: [] for m in modes}
    for _ in range(steps):
        for m in modes:
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            handles[m].collect_eig_batched(batch)
            torch.cuda.synchronize()
            wall[m].append((time.perf_counter() - t0) * 1000.0)
            kern[m].append(handles[m].timings())
    out = {}
    sel_d = torch.as_tensor(sel, device=ctx.device)
    for m in modes:
        h = handles[m]
        h.sync()
        h.reset()
        h.collect_eig_batched(batch)
        h.sync()
        sampled = h.images[0][:, sel_d].double().cpu().numpy()
        h.close()
        ms = float(np.mean(wall[m]))
        stage = float(np.mean([k[1] for k in kern[m]]))
        synth = float(np.mean([k[2] for k in kern[m]]))
        log(f"{m}: {ms:.1f} ms/step, synthesis kernel {synth:.1f} ms, staging {stage:.2f} ms")
        out[m] = (ms, synth, stage, batch.products, sampled, tune.get(m))
    return out


def level_errors(got, want):
    """Per level: max |I - I_ref| / max |I_ref| and rms(I - I_ref) / rms(I_ref) (levels with I_ref = 0 skipped)."""
    mx, rms = [], []
    for a, b in zip(np.asarray(got, np.float64), np.asarray(want, np.float64)):
        if np.max(np.abs(b)) == 0:
            continue
        mx.append(float(np.max(np.abs(a - b)) / np.max(np.abs(b))))
        rms.append(float(np.sqrt(np.mean((a - b) ** 2) / np.mean(b * b))))
    return mx, rms


def oracle_leg(items, pix, n_levels, workers):
    """The FP64 oracle over every epoch of a workload at the pixels ``pix`` (the CPU-baseline leg).

    Independent epochs run on ``workers`` host threads, each calling the
    oracle's BLAS evaluator with one BLAS thread (its exponentials and
    products release the interpreter lock); the eigenpairs are the ones the
    GPU launch used (W rounded to complex64, weights to float32, as the
    library reads them).  Returns (images (n_levels, n_pix) summed over
    epochs, wall seconds, products).
    """
    import concurrent.futures as cf
    import oracle as ref
    from threadpoolctl import threadpool_limits

    def host(a):
        return a.cpu().numpy() if hasattr(a, "cpu") else np.asarray(a)

    work = [(x, wl, host(W).astype(np.complex64).astype(np.complex128),
             host(d).astype(np.float32).astype(np.float64), host(lev)) for _, x, wl, W, d, lev in items]

    def one(item):
        x, wl, Wn, dn, ln = item
        member = ref.membership_from_level_of(ln, n_levels)
        return ref.synthesize_blas(Wn, dn, member, x, pix, wl), x.shape[0] * int((ln >= 0).sum())

    t0 = time.perf_counter()
    with threadpool_limits(limits=1):
        with cf.ThreadPoolExecutor(max_workers=workers) as ex:
            res = list(ex.map(one, work))
    dt = time.perf_counter() - t0
    img = np.sum([r[0] for r in res], axis=0)
    prods = float(sum(r[1] for r in res)) * pix.shape[0]
    return img, dt, prods


def host_workers():
    """Host threads for the oracle leg: the cores this process may run on, at most 16."""
    return max(1, min(16, len(os.sched_getaffinity(0))))


def measure_c4(args, torch, ctx):
    """Batched uneven instances (a6): 64 channels x 32 epochs, L 200..512, K 16..128, 512^2 pixels, one call."""
    from paper_2310_09200_amd import Batch, StandardSynthesis
    from sims import configs
    w = configs.c4()
    items = []
    for i in range(w.n_instances()):
        inst = w.instance(i)
        items.append((inst.slot, inst.x, inst.wl, inst.W.astype(np.complex64), inst.lam.astype(np.float32),
                      inst.level_of))
    batch = Batch(items, ctx.device)
    s = StandardSynthesis(ctx, w.pix, 4, 64, 512, 128, args.precision)
    tune = None
    if args.c4_tiles:
        s.tiles = [int(v) for v in args.c4_tiles.split(",")]
        log(f"C4: tiles {s.tiles} as given")
    elif not args.no_autotune:
        t0 = time.perf_counter()
        table = s.autotune_batched(batch, reps=1)
        tune = {"tiles": s.tiles, "ms_per_launch_by_class_and_tile": table, "seconds": time.perf_counter() - t0}
        log(f"C4: autotuned tiles {s.tiles} from {table}")
    s.collect_eig_batched(batch)
    torch.cuda.synchronize()
    ms = []
    for _ in range(max(1, args.steps)):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        s.collect_eig_batched(batch)
        torch.cuda.synchronize()
        ms.append((time.perf_counter() - t0) * 1000.0)
    kern = s.timings()[2]
    s_tiles = s.tiles
    s.close()
    prods = batch.products * w.n_pix
    log(f"C4 batched: {np.mean(ms):.1f} ms/call, synthesis {kern:.1f} ms, {prods / (np.mean(ms) / 1e3):.3e} products/s")
    return {"workload": "2048 uneven instances (64 channels x 32 epochs, L 200..512, K 16..128, 4 levels), "
                        "512x512 pixels, one batched call", "contraction": args.precision,
            "products": prods, "ms_per_call": float(np.mean(ms)), "synthesis_kernels_ms": kern, "autotune": tune,
            "tiles": s_tiles,
            "value": prods / (np.mean(ms) / 1e3), "unit": "products/s",
            "algorithmic_fp32_rate_over_peak": ALG_FLOP * prods / (np.mean(ms) / 1e3) / (FP32_PEAK_TFLOPS * 1e12),
            "mfma_fraction_of_own_peak": EXEC_FLOP[args.precision] * prods / (kern / 1e3) / (PEAK[args.precision] * 1e12)}


def measure_c5_backward(args, torch, ctx):
    """Backward (a7): L=256, K=64, 512^2 pixels, 4 levels; forward image and gradients w.r.t. W, d, x."""
    from paper_2310_09200_amd import StandardSynthesis
    from sims import configs
    from sims.levels import kmeans1d_intervals
    w = configs.c5()
    inst = w.instance(0)
    s = StandardSynthesis(ctx, w.pix, 4, 1, 256, 64, "fp32")
    probe = StandardSynthesis(ctx, w.pix[:1], 1, 1, 256, 256)
    _, lam, _, _ = probe.prestep(inst.x, inst.wl, inst.V, 64, np.array([[-np.inf, np.inf]]))
    probe.close()
    iv = kmeans1d_intervals(lam.cpu().numpy(), 4, negative_level=False)
    W, lam, d, lev = s.prestep(inst.x, inst.wl, inst.V, 64, iv)
    gimg = torch.as_tensor(w.meta["loss_weights"](), dtype=torch.float32, device=ctx.device)
    s.eig_backward(inst.x, inst.wl, W, d, lev, gimg)
    s.collect_eig(0, inst.x, inst.wl, W, d, lev)
    torch.cuda.synchronize()
    fwd, bwd = [], []
    for _ in range(5):
        s.collect_eig(0, inst.x, inst.wl, W, d, lev)
        fwd.append(s.timings()[2])
        s.eig_backward(inst.x, inst.wl, W, d, lev, gimg)
        bwd.append(s.timings()[2])
    s.close()
    # the same array and pixels with 128 eigenpairs: the two-kernel backward (two eigenpair slices per chunk)
    s2 = StandardSynthesis(ctx, w.pix, 4, 1, 256, 128, "fp32")
    probe = StandardSynthesis(ctx, w.pix[:1], 1, 1, 256, 256)
    _, lam128, _, _ = probe.prestep(inst.x, inst.wl, inst.V, 128, np.array([[-np.inf, np.inf]]))
    probe.close()
    iv2 = kmeans1d_intervals(lam128.cpu().numpy(), 4, negative_level=False)
    W2, lam2, d2, lev2 = s2.prestep(inst.x, inst.wl, inst.V, 128, iv2)
    kept2 = int((lev2 >= 0).sum().item())
    s2.eig_backward(inst.x, inst.wl, W2, d2, lev2, gimg)
    torch.cuda.synchronize()
    bwd2 = []
    for _ in range(5):
        s2.eig_backward(inst.x, inst.wl, W2, d2, lev2, gimg)
        bwd2.append(s2.timings()[2])
    s2.close()
    prods = 256 * int((lev >= 0).sum().item()) * w.n_pix  # kept eigenpairs (all 64 when every one is in a level)
    f_ms, b_ms, b2_ms = float(np.median(fwd)), float(np.median(bwd)), float(np.median(bwd2))
    log(f"C5: forward {f_ms:.3f} ms, backward {b_ms:.3f} ms; K = 128 backward {b2_ms:.3f} ms ({kept2} kept)")
    return {"workload": "L=256, K=64, 512x512 pixels, 4 levels, loss weights N(0,1) per level and pixel",
            "forward_ms": f_ms, "backward_ms": b_ms, "products": prods,
            "k128_backward_ms": b2_ms, "k128_kept_eigenpairs": kept2,
            "k128_backward_fp32_mfma_fraction": 14.0 * 256 * kept2 * w.n_pix / (b2_ms / 1e3) / (FP32_PEAK_TFLOPS * 1e12),
            "backward_note": "E recompute (FP32 MFMA, three products) + dd/M, dW = 2 B M^T on split fp16 products and "
                             "H = conj(W) M on FP32 MFMA -> dx; three times the forward's complex MACs, executed as "
                             "6 + 8 FP32 and 24 fp16 flop per product; the fraction counts the 14 FP32 ones",
            "backward_fp32_mfma_fraction": 14.0 * prods / (b_ms / 1e3) / (FP32_PEAK_TFLOPS * 1e12)}


def measure_nufft(args, torch, ctx):
    """NUFFT synthesis next to standard synthesis on the paper's performance setup.

    SKA-Low-like array (C3: 512 stations, 65 km), 50 epochs over 6 h, 4 arcsec
    pixels, 8 + 1 k-means levels, every eigenpair kept; eigenpairs from the GPU
    FP64 pre-step.  Both syntheses image the same eigenpairs; the NUFFT image
    is compared with the standard one level by level.
    """
    from paper_2310_09200_amd import Batch, NufftSynthesis, StandardSynthesis
    from sims import configs, tangent_basis
    from sims.levels import kmeans1d_intervals
    side = args.nufft_side
    fov = side * 4.0 / 3600.0
    w = configs.c3(n_steps=50, n_side=side, fov_deg=fov)
    insts = [w.instance(i) for i in range(w.n_steps)]
    probe = StandardSynthesis(ctx, w.pix[:1], 1, 1, 512, 512)
    _, lam0, _, _ = probe.prestep(insts[0].x, insts[0].wl, insts[0].V, 512, np.array([[-np.inf, np.inf]]))
    probe.close()
    iv = kmeans1d_intervals(lam0.cpu().numpy(), 8, negative_level=True)
    n_levels = iv.shape[0]
    pre = StandardSynthesis(ctx, w.pix[:1], n_levels, 1, 512, 512)
    items = []
    for inst in insts:
        W, lam, d, lev = pre.prestep(inst.x, inst.wl, inst.V, 512, iv)
        items.append((0, inst.x, inst.wl, W.clone(), d.clone(), lev.clone()))
    pre.close()
    batch = Batch(items, ctx.device)
    frame = np.array(tangent_basis(w.dec0_deg))
    uvw = np.zeros(3)
    for inst in insts:
        li, mi = np.triu_indices(inst.x.shape[0], k=1)
        b = (inst.x[li] - inst.x[mi]) @ frame.T / inst.wl
        uvw = np.maximum(uvw, np.max(np.abs(b), axis=0))
    uvw = uvw * 1.001

    s = StandardSynthesis(ctx, w.pix, n_levels, 1, 512, 512, args.precision)
    plan = NufftSynthesis(ctx, w.pix, n_levels, 512, 512, args.nufft_eps, frame, uvw, transform=args.nufft_transform,
                          partitions=args.nufft_partitions, uvw_partitions=args.nufft_uvw_partitions)
    N, M, kw = plan.shape
    s.collect_eig_batched(batch)
    plan.collect_eig_batched(batch)
    plan.emit()
    torch.cuda.synchronize()
    s.reset()
    plan.images.zero_()
    std_ms, nu_ms, spread_ms, emit_ms = [], [], [], []
    for _ in range(max(1, args.steps)):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        s.collect_eig_batched(batch)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        plan.collect_eig_batched(batch)
        plan.emit()
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        std_ms.append((t1 - t0) * 1e3)
        nu_ms.append((t2 - t1) * 1e3)
        a, b = plan.timings()
        spread_ms.append(a)
        emit_ms.append(b)
    plan.sync()
    s.sync()
    std_img = s.images[0].double()
    nu_img = plan.images.double()
    errs = []
    for lv in range(n_levels):
        peak = float(std_img[lv].abs().max())
        if peak > 0:
            errs.append(float((nu_img[lv] - std_img[lv]).abs().max()) / peak)
    s.close()
    plan.close()
    prods = batch.products * w.n_pix
    log(f"NUFFT {side}^2 ({args.nufft_partitions}x{args.nufft_partitions} image, {args.nufft_uvw_partitions}x"
        f"{args.nufft_uvw_partitions} uvw partitions): standard {np.mean(std_ms):.1f} ms, NUFFT {np.mean(nu_ms):.1f} ms "
        f"(spread {np.mean(spread_ms):.1f}, emit {np.mean(emit_ms):.1f}), grid {N} fft {M} w={kw}, "
        f"max level diff {max(errs):.2e}")
    return {"workload": f"SKA-Low-like 512 stations (65 km), 50 epochs over 6 h, {side}x{side} pixels of 4 arcsec "
                        f"({fov * 60:.1f} arcmin), 8+1 k-means levels, all 512 eigenpairs (GPU FP64 pre-step)",
            "epsilon": args.nufft_eps, "spread_grid": list(N), "fft_grid": list(M), "kernel_width": kw,
            "standard_ms": float(np.mean(std_ms)), "standard_contraction": args.precision,
            "nufft_ms": float(np.mean(nu_ms)), "nufft_spread_ms": float(np.mean(spread_ms)),
            "nufft_emit_ms": float(np.mean(emit_ms)), "speedup_nufft_over_standard": float(np.mean(std_ms) / np.mean(nu_ms)),
            "products": prods, "standard_products_per_s": prods / (np.mean(std_ms) / 1e3),
            "partitions": args.nufft_partitions, "uvw_partitions": args.nufft_uvw_partitions,
            "transform": {"auto": "pruned, own LDS line FFTs where every axis fits (a direct DFT on MFMA for axes of at most 64 points), else rocFFT",
                          "rocfft": "pruned, rocFFT"}[args.nufft_transform],
            "max_level_diff_nufft_vs_standard": max(errs)}


def measure_nufft_memory(args, torch, ctx):
    """Device memory of NUFFT plans for the widest field here (the SKA-Low-like C3 field: 8 deg, 2048^2 pixels,
    65 km baselines over 50 epochs, 8+1 levels, eps 1e-5), one grid against image x uvw partitions (Section 3.4.1).

    Partitioned plans: bb_nufft_workspace_size of the library (one shared grid and transform buffers for the
    largest (tile, cell) pair, plus each tile's tables, pixels and images).  One grid: its n_levels N0 N1 N2
    complex64 cells from the same grid rules (the pruned transform's stage buffers come on top).
    """
    import ctypes
    from paper_2310_09200_amd import _lib
    from sims import configs, tangent_basis
    from oracle import nufft_ref
    w = configs.c3(n_steps=50, n_side=2048)
    frame = np.array(tangent_basis(w.dec0_deg))
    uvw = np.zeros(3)
    for i in range(w.n_steps):
        inst = w.instance(i)
        li, mi = np.triu_indices(inst.x.shape[0], k=1)
        uvw = np.maximum(uvw, np.max(np.abs((inst.x[li] - inst.x[mi]) @ frame.T / inst.wl), axis=0))
    uvw = uvw * 1.001
    n_levels, eps = 9, 1e-5
    N = nufft_ref.plan_params(eps, uvw, nufft_ref.rotate(w.pix, frame))["N"]
    one_grid = 8.0 * float(np.prod(N)) * n_levels
    pix_cm = np.ascontiguousarray(np.asarray(w.pix, np.float64).T)
    out = {"workload": "SKA-Low-like 512 stations (65 km), 50 epochs, 2048x2048 pixels over 8 deg, 8+1 levels, "
                       "eps 1e-5",
           "uvw_max": list(uvw), "one_grid": {"spread_grid": [int(n) for n in N], "grid_bytes": one_grid,
                                              "source": "grid rules (oracle plan_params)"},
           "partitioned": []}
    log(f"NUFFT memory, 8 deg 2048^2 field: one grid {N} = {one_grid / 1e9:.0f} GB of grid cells")
    for P, Q in [(8, 1), (8, 2), (8, 4)]:
        opt = _lib.bb_nufft_options(n_levels=n_levels, n_ant_max=512, k_max=512, transform=0, epsilon=eps,
                                    partitions=P, uvw_partitions=Q)
        fr = frame.reshape(9)
        for i in range(9):
            opt.frame[i] = float(fr[i])
        for i in range(3):
            opt.uvw_max[i] = float(uvw[i])
        sz = ctypes.c_size_t()
        st = ctx.lib.bb_nufft_workspace_size(ctx.handle, ctypes.byref(opt), pix_cm.shape[1],
                                             ctypes.c_void_p(pix_cm.ctypes.data), ctypes.byref(sz))
        rec = {"partitions": P, "uvw_partitions": Q, "status": _lib.STATUS.get(st, st),
               "workspace_bytes": int(sz.value) if st == 0 else None, "source": "bb_nufft_workspace_size"}
        out["partitioned"].append(rec)
        log(f"NUFFT memory, {P}x{P} image x {Q}x{Q} uvw partitions: "
            f"{(sz.value / 1e9) if st == 0 else float('nan'):.1f} GB workspace")
    return out


def measure_workload(args, torch, ctx, w, items, n_levels, modes, sel, steps, warmup, workers):
    """Time every mode on one batched workload and check the timed launch against the oracle.

    Returns (per-mode dict, oracle-leg record, timing tuple of the first mode).
    """
    timing = time_modes(args, torch, ctx, w, items, modes, n_levels, sel, steps, warmup)
    ref_img, dt, oprods = oracle_leg(items, w.pix[sel], n_levels, workers)
    out = {}
    for m in modes:
        ms_m, kern_m, stage_m, prods_m, sampled, tune_m = timing[m]
        total = prods_m * w.n_pix
        mx, rms = level_errors(sampled, ref_img)
        out[m] = {"value": total / (ms_m / 1e3), "ms_per_step": ms_m, "kernel_ms": kern_m,
                  "algorithmic_fp32_rate_over_peak": ALG_FLOP * total / (kern_m / 1e3) / (FP32_PEAK_TFLOPS * 1e12),
                  "mfma_fraction_of_own_peak": EXEC_FLOP[m] * total / (kern_m / 1e3) / (PEAK[m] * 1e12),
                  "level_max_rel_error": mx, "level_rms_rel_error": rms, "max_level_error": max(mx),
                  "autotune": tune_m}
        log(f"  {m}: per-level max error vs oracle {max(mx):.2e}, rms {max(rms):.2e}")
    leg = {"seconds": dt, "products": oprods, "value": oprods / dt, "pixels": int(len(sel)),
           "epochs": len(items)}
    return out, leg, timing


def measure_c1(args, torch, ctx, modes, workers):
    """C1: 64 antennas in a 2 km disk, 128^2 pixels over 5 deg, 1 epoch, 4 + 1 levels; single-instance call."""
    from paper_2310_09200_amd import StandardSynthesis
    from sims import configs
    w = configs.c1()
    inst = w.instance(0)
    _, items, pre_ms = gpu_eigenpairs(torch, ctx, w, [inst], 64, 4)
    _, x, wl, W, d, lev = items[0]
    ref_img, dt, oprods = oracle_leg(items, w.pix, 5, workers)
    x = torch.as_tensor(x).to(ctx.device)  # inputs resident on the device, as in the timed batched launches
    prods = float(x.shape[0]) * int((lev >= 0).sum().item()) * w.n_pix
    out = {}
    for m in modes:
        s = StandardSynthesis(ctx, w.pix, 5, 1, 64, 64, m)
        for _ in range(3):
            s.collect_eig(0, x, wl, W, d, lev)
        torch.cuda.synchronize()
        kern, wall = [], []
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            s.collect_eig(0, x, wl, W, d, lev)
            torch.cuda.synchronize()
            wall.append((time.perf_counter() - t0) * 1e3)
            kern.append(s.timings()[2])
        s.reset()
        s.collect_eig(0, x, wl, W, d, lev)
        s.sync()
        got = s.images[0].double().cpu().numpy()
        s.close()
        mx, rms = level_errors(got, ref_img)
        k_ms, w_ms = float(np.median(kern)), float(np.median(wall))
        out[m] = {"value": prods / (w_ms / 1e3), "ms_per_call": w_ms, "kernel_ms": k_ms,
                  "kernel_products_per_s": prods / (k_ms / 1e3),
                  "level_max_rel_error": mx, "level_rms_rel_error": rms, "max_level_error": max(mx)}
        log(f"C1 {m}: {w_ms:.3f} ms per call (kernel {k_ms:.3f} ms), max level error {max(mx):.2e}")
    return {"workload": "C1: 64 antennas in a 2 km disk, 128x128 pixels over 5 deg, 1 epoch at 150 MHz, "
                        "all 64 eigenpairs in 4+1 k-means levels; one single-instance call, median of 20",
            "products": prods, "unit": "products/s", "prestep_ms": pre_ms["single_call_ms_per_epoch"], "modes": out,
            "error_reference": "FP64 oracle, full image"}


def measure_c3(args, torch, ctx, modes, workers):
    """C3: SKA-Low-like precision study and throughput at 2048^2, 50 epochs (the paper's performance shape)."""
    from sims import configs
    w = configs.c3(n_steps=50, n_side=2048)
    t0 = time.time()
    insts = [w.instance(i) for i in range(w.n_steps)]
    log(f"C3: simulated {len(insts)} visibility matrices in {time.time() - t0:.1f}s")
    iv, items, pre_ms = gpu_eigenpairs(torch, ctx, w, insts, 512, 8)
    n_levels = iv.shape[0]
    sel = sims_sample(w)
    out, leg, timing = measure_workload(args, torch, ctx, w, items, n_levels, modes, sel,
                                        steps=max(1, min(args.steps, 2)), warmup=1, workers=workers)
    comp = {}
    for cm in ("bf16x3", "bf16x3_3m"):
        for pm in ("fp32", "fp32_3m"):
            if cm in out and pm in out:
                comp[f"speedup_{cm}_over_{pm}"] = out[pm]["ms_per_step"] / out[cm]["ms_per_step"]
    first = modes[0]
    log(f"C3: {out[first]['value']:.3e} products/s ({first}); oracle leg {leg['seconds']:.1f}s")
    return {"workload": "C3: SKA-Low-like 512 stations (65 km), 2048x2048 pixels over 8 deg, 50 epochs over 6 h at "
                        "150 MHz, all 512 eigenpairs in 8+1 k-means levels; one batched launch over all epochs",
            "products": timing[first][3] * w.n_pix, "unit": "products/s", "value": out[first]["value"],
            "contraction": first, "prestep_ms_per_epoch": pre_ms["batched_ms_per_epoch"], "modes": out,
            "compensated_vs_fp32": comp,
            "error_reference": f"FP64 oracle summed over all {leg['epochs']} epochs at {leg['pixels']} pixels "
                               "(every 8th row and column, 9x9 around each source, last pixel)",
            "oracle_leg": leg}


def sims_sample(w):
    import sims
    return sims.sample_pixels(w.n_side, w.source_pixels(), stride=8)


MODES = ("fp32_3m", "fp32", "bf16x3", "bf16x3_3m")
# executed MFMA work per product: 8 flop (four real MACs) or 6 (three), each as three products of split
# 16-bit words (fp16 hi + lo in the FP32 modes, bf16 hi + lo in the BF16 modes)
EXEC_FLOP = {"fp32": 24.0, "fp32_3m": 18.0, "bf16x3": 24.0, "bf16x3_3m": 18.0}
PEAK = {m: F16_PEAK_TFLOPS for m in MODES}
# the metric's own unit: one product is one complex MAC, 8 real flop
ALG_FLOP = 8.0


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--precision", default="fp32_3m", choices=MODES,
                    help="contraction of the headline line: fp32_3m (FP32, three real products per complex "
                         "product), fp32 (FP32, four), bf16x3 (BF16 hi/lo, three bf16 products per real product, "
                         "four real products), bf16x3_3m (BF16 hi/lo, three real products)")
    ap.add_argument("--epochs", type=int, default=100)
    ap.add_argument("--n-side", type=int, default=1024)
    ap.add_argument("--no-cpu-baseline", action="store_true",
                    help="skip the oracle leg (CPU baseline and the error check of the timed launches)")
    ap.add_argument("--no-compare", action="store_true", help="time only the headline contraction mode")
    ap.add_argument("--no-extra", action="store_true",
                    help="skip the C1, C3, batched (C4), backward (C5) and NUFFT-synthesis measurements")
    ap.add_argument("--nufft-side", type=int, default=1024, help="image side of the NUFFT comparison (4 arcsec pixels)")
    ap.add_argument("--nufft-eps", type=float, default=1e-5)
    ap.add_argument("--nufft-transform", choices=["auto", "rocfft"], default="auto",
                    help="type-2 transform of the NUFFT comparison")
    ap.add_argument("--nufft-partitions", type=int, default=1,
                    help="image-domain partitions per axis of the NUFFT comparison")
    ap.add_argument("--nufft-uvw-partitions", type=int, default=1,
                    help="uvw-domain partitions per axis of the NUFFT comparison")
    ap.add_argument("--only-nufft", action="store_true",
                    help="print only the NUFFT-vs-standard measurement (for profiling it alone)")
    ap.add_argument("--only-c4", action="store_true",
                    help="print only the batched uneven-instance measurement (for profiling it alone)")
    ap.add_argument("--c4-tiles", default=None,
                    help="tile ids per K class for the batched uneven-instance measurement, comma-separated "
                         "(-1 keeps a class's default); implies no autotuning there")
    ap.add_argument("--no-autotune", action="store_true",
                    help="keep the default tile shapes instead of timing the candidates before the timed steps")
    ap.add_argument("--calibration-copy-mb", type=int, default=0,
                    help="before timing, copy this many MiB device-to-device once (a kernel of known traffic "
                         "for scaling hardware byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU: this build has no multi-GPU path (instances or pixel tiles would be "
              "sharded across GPUs with one final all-reduce of the images). Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)
    import torch
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(2)
    dev = torch.device("cuda", 0)

    if args.calibration_copy_mb > 0:
        n = args.calibration_copy_mb * (1 << 20) // 4
        src = torch.ones(n, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        log(f"calibration copy: {args.calibration_copy_mb} MiB read + {args.calibration_copy_mb} MiB written")
        del src, dst
    if args.only_nufft:
        from paper_2310_09200_amd import Context
        print(json.dumps({"nufft_vs_standard": measure_nufft(args, torch, Context(0))}), flush=True)
        return
    if args.only_c4:
        from paper_2310_09200_amd import Context
        print(json.dumps({"batched_c4": measure_c4(args, torch, Context(0))}), flush=True)
        return
    ctx, w, intervals, items, insts, pre_ms = build_inputs(args, torch, dev)
    n_levels = intervals.shape[0]
    modes = [args.precision] + ([] if args.no_compare else [m for m in MODES if m != args.precision])
    workers = host_workers()
    sel = sims_sample(w)

    timing = time_modes(args, torch, ctx, w, items, modes, n_levels, sel)
    ms, kern, stage, products, _, _ = timing[args.precision]
    total_products = products * w.n_pix
    value = total_products / (ms / 1000.0)

    flops = EXEC_FLOP[args.precision] * total_products
    achieved = flops / (kern / 1000.0) / 1e12
    counters = counter_figures(args.precision)
    traffic = None
    if counters and "fetch_bytes" in counters and "write_bytes" in counters:
        traffic = counters["fetch_bytes"] + counters["write_bytes"]
    out = {
        "metric": "pixel*antenna*eigvec products/s for standard synthesis; compensated vs plain FP32 at 1e-4",
        "value": value,
        "unit": "products/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16x3" if args.precision.startswith("bf16") else "f32 (fp16 hi+lo operands, f32 accumulators)",
        "data": "synthetic",
        "config": {"workload": f"LOFAR-like single channel: L=512 stations (50 km), K=512 eigenpairs, "
                               f"{w.n_side}x{w.n_side} pixels over 10 deg, {args.epochs} epochs over 6 h, "
                               f"{n_levels - 1}+1 k-means levels, FP64 phase arguments",
                   "n_ant": 512, "n_eig": 512, "n_pix": w.n_pix, "n_instances": args.epochs,
                   "n_levels": n_levels, "contraction": args.precision,
                   "launch": "batched: one synthesis launch over all epochs per step"},
        "algorithmic_fp32_rate_over_peak": ALG_FLOP * value / (FP32_PEAK_TFLOPS * 1e12),
        "algorithmic_fp32_rate_note": "8 flop per product (one complex MAC as four real MACs) x products/s / "
                                      "157.3 TFLOP/s FP32 matrix peak: the FP32-equivalent rate the >= 50 % target "
                                      "is stated in; above 1 because the products run as three 16-bit products of "
                                      "split words (fp16 hi + lo: images closer to 64 bits than with FP32 MFMAs). "
                                      "roofline.frac is the executed-flop fraction of the 16-bit matrix peak.",
        "kernel_ms_per_step": kern,
        "staging_ms_per_step": stage,
        "prestep_ms_per_epoch": pre_ms["batched_ms_per_epoch"],
        "prestep": pre_ms,
        "prestep_note": "FP64 Gram + rocSOLVER strided-batched zhegvd + selection for all epochs in one library call "
                        "(bb_synth_prestep_batched, one host wait), wall clock per epoch; single_call is one "
                        "bb_synth_prestep call per epoch. Not in the metric (the synthesis of one epoch takes "
                        "kernel_ms_per_step / epochs)",
        "roofline": {"bound": "mfma", "achieved": achieved, "peak": PEAK[args.precision], "unit": "TFLOP/s",
                     "frac": achieved / PEAK[args.precision], "traffic": traffic,
                     "kernel": "synth_fwd_kernel",
                     "flops_per_launch": flops,
                     "flop_per_product": EXEC_FLOP[args.precision]},
    }
    if counters and "mfma_busy" in counters:
        out["roofline"]["mfma_busy_counter"] = counters["mfma_busy"]
    # phase generation (FP64 argument and reduction, hardware sin/cos) against its own peak on this device:
    # the synthesis kernel evaluates every phase once per K pass of its tile (256 eigenpairs for K > 128)
    peak_pairs, probe_ms, probe_pairs = measure_phase_peak(torch, ctx, w, items)
    n_ant, n_eig, eig_per_pass = 512, 512, 256
    n_pass = -(-n_eig // eig_per_pass)
    alg_pairs = float(n_ant) * w.n_pix * args.epochs
    gen_pairs = n_pass * alg_pairs
    pg = {
        "peak_pairs_per_s": peak_pairs, "probe": f"bb_phase_probe: {probe_pairs:.3e} pairs in {probe_ms:.3f} ms",
        "pairs_per_launch": alg_pairs, "passes": n_pass,
        "achieved_pairs_per_s": alg_pairs / (kern / 1000.0),
        "frac": alg_pairs / (kern / 1000.0) / peak_pairs,
        "generated_frac": gen_pairs / (kern / 1000.0) / peak_pairs,
        "note": "pairs_per_launch = N_pix * L * epochs; generated_frac counts every pass's evaluation: the share "
                "of the launch that phase generation would take at its own peak"}
    probe_c = counter_figures("probe")
    if counters and probe_c and "trans_instructions" in counters and "trans_instructions" in probe_c:
        synth_rate = counters["trans_instructions"] / (kern / 1e3)
        probe_rate = probe_c["trans_instructions"] / (probe_ms / 1e3)
        pg["counter"] = {"synth_trans_wave_instructions_per_launch": counters["trans_instructions"],
                         "probe_trans_wave_instructions_per_call": probe_c["trans_instructions"],
                         "synth_sincos_per_s": 64.0 * synth_rate, "probe_sincos_per_s": 64.0 * probe_rate,
                         "sincos_throughput_frac": synth_rate / probe_rate,
                         "note": "transcendental (sin, cos) wave instructions from rocprofv3 SQ_INSTS_VALU_TRANS_F32 "
                                 "over this run's HIP-event kernel times; the probe is the device's peak for phase "
                                 "generation alone"}
    out["phase_generation"] = pg
    log(f"phase generation: probe peak {peak_pairs:.3e} pairs/s; synthesis {alg_pairs / (kern / 1000.0):.3e} "
        f"pairs/s ({100 * alg_pairs / (kern / 1000.0) / peak_pairs:.1f} % of peak; with {n_pass} passes "
        f"{100 * gen_pairs / (kern / 1000.0) / peak_pairs:.1f} %)")
    modes_out = {}
    for m in modes:
        ms_m, kern_m, _, _, _, tune_m = timing[m]
        modes_out[m] = {"value": total_products / (ms_m / 1000.0), "ms_per_step": ms_m, "kernel_ms": kern_m,
                        "autotune": tune_m,
                        "algorithmic_fp32_rate_over_peak": ALG_FLOP * total_products / (kern_m / 1000.0)
                        / (FP32_PEAK_TFLOPS * 1e12),
                        "mfma_fraction_of_own_peak": EXEC_FLOP[m] * total_products / (kern_m / 1000.0)
                        / (PEAK[m] * 1e12)}
        cm = counter_figures(m)
        if cm and "mfma_busy" in cm:
            modes_out[m]["mfma_busy_counter"] = cm["mfma_busy"]
    out["modes"] = modes_out
    comp = {}
    for cm in ("bf16x3", "bf16x3_3m"):
        for pm in ("fp32", "fp32_3m"):
            if cm in timing and pm in timing:
                comp[f"speedup_{cm}_over_{pm}"] = timing[pm][0] / timing[cm][0]
    if comp:
        out["compensated_vs_fp32"] = comp
    if not args.no_cpu_baseline:
        # the oracle leg: FP64 reference of the timed launch's own images (all epochs, sampled pixels),
        # timed on the host's cores -> the CPU baseline and the per-level errors of every mode
        ref_img, dt, oprods = oracle_leg(items, w.pix[sel], n_levels, workers)
        log(f"oracle: {len(sel)} pixels x {len(items)} epochs in {dt:.1f}s -> {oprods / dt:.3e} products/s on "
            f"{workers} threads")
        out["cpu_baseline"] = {"value": oprods / dt, "unit": "products/s", "cores": workers, "kind": "oracle",
                               "sample": f"all {len(items)} epochs at {len(sel)} of the {w.n_pix} pixels (every 8th "
                                         f"row and column, the 9x9 neighbourhood of each of the "
                                         f"{len(w.source_pixels())} point sources, the last pixel); L=512, K=512, "
                                         f"FP64 numpy/BLAS, one epoch per host thread, {dt:.1f} s",
                               "affinity_cores": len(os.sched_getaffinity(0))}
        errs = {}
        for m in modes:
            mx, rms = level_errors(timing[m][4], ref_img)
            errs[m] = {"level_max_rel_error": mx, "level_rms_rel_error": rms, "max": max(mx), "rms": max(rms)}
            log(f"{m}: timed launch vs oracle, per-level max {max(mx):.2e}, rms {max(rms):.2e}")
        out["max_level_error_vs_oracle"] = {m: errs[m]["max"] for m in modes}
        out["error_vs_oracle"] = {
            "reference": "the timed launch itself (reset, one batched launch over all epochs) against the FP64 "
                         "oracle summed over the same epochs and eigenpairs, at the cpu_baseline sample pixels",
            "definition": "per level max|I - I_ref| / max|I_ref| and rms(I - I_ref) / rms(I_ref)",
            "modes": errs}
    if not args.no_extra:
        out["c1"] = measure_c1(args, torch, ctx, modes, workers)
        if not args.no_cpu_baseline:
            out["c3"] = measure_c3(args, torch, ctx, modes, workers)
        out["batched_c4"] = measure_c4(args, torch, ctx)
        out["backward_c5"] = measure_c5_backward(args, torch, ctx)
        out["nufft_vs_standard"] = measure_nufft(args, torch, ctx)
        out["nufft_memory"] = measure_nufft_memory(args, torch, ctx)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
