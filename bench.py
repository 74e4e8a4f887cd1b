"""Throughput benchmark of the Drude-FDTD forward + adjoint + gradient hot path.

One step = set_density (device tensor) + forward solve + adjoint solve +
gradient (device tensor) of one seeded density, i.e. one topology-optimization
iteration.  The default workload is the 3D FP32 case: 256^3 Yee grid, dx =
2 nm, 16-cell CPML, 128 x 128 x 32 design slab, 4^3 gap, x-polarized plane
wave along +z, 8000 steps, 16 DFT frequencies over 600-900 nm.  The 2D TMz
FP32 case (--workload c2: 2048^2 grid, 512^2 design box, 5 x 5 gap, 20000
steps, 16 frequencies over 500-1000 nm) cycles the collision-rate multiplier
through {1, 4, 16} (damping continuation).

Prints ONE JSON line: the metric in Gcell-updates/s (grid cells x time steps x
2 solves / wall time of the step), the roofline of the time-step kernel
(algorithmic HBM bytes per time step / average time per step from HIP events on the
library stream), and the CPU oracle timed on a bounded sample of the same
workload on the host cores.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

import fdtd_workloads as W  # noqa: E402

METRIC = "Drude-FDTD fwd+adjoint Gcell-updates/s, % HBM roofline; time-to-design vs plain"
HBM_PEAK_GBS = 8000.0

# HBM bytes per time step of the step kernels from rocprofv3 FETCH_SIZE / WRITE_SIZE
# passes (scaled by the copy-probe factors: fetch x2, write x1), recorded with
# the sources they were taken on: the kernels and the library code that
# orders their workgroups.  Reported only while those sources are unchanged;
# the summaries live in profiles/.
SRC_2D = ["paper_2203_01462_amd/csrc/fdtd_2d_multi.hip", "paper_2203_01462_amd/csrc/fdtd_multi.hpp", "paper_2203_01462_amd/csrc/fdtd_api.hip"]
SRC_BATCH = ["paper_2203_01462_amd/csrc/fdtd_2d.hip", "paper_2203_01462_amd/csrc/fdtd_api.hip"]
SRC_3D = ["paper_2203_01462_amd/csrc/fdtd_3d.hip", "paper_2203_01462_amd/csrc/fdtd_api.hip"]
SRC_TE = ["paper_2203_01462_amd/csrc/fdtd_te_multi.hip", "paper_2203_01462_amd/csrc/fdtd_multi.hpp", "paper_2203_01462_amd/csrc/fdtd_api.hip"]
MEASURED_TRAFFIC = {
    # one launch = eight time steps of the grid
    "tmz2d_2048_fp32": {"sources": SRC_2D, "sha256_16": "f3d92ea55c2a1435",
                        "fwd": 26.5e6, "adj": 29.4e6,
                        "profile": "profiles/step2d_multi_tmz2d_2048_fp32.md"},
    # one time step of all 64 instances = one step2d_batch_mix_kernel launch
    "tmz2d_batch64_c4": {"sources": SRC_BATCH, "sha256_16": "533bf3d697cc0670",
                         "fwd": 500.2e6, "adj": 521.8e6,
                         "profile": "profiles/step2d_batch_mix_kernel_tmz2d_batch64_c4.md"},
    # one time step = the general update (forward: one step3d_general_fwd
    # launch; adjoint: three step3d_general launches) + step3d_plain
    "yee3d_256_fp32": {"sources": SRC_3D, "sha256_16": "4973fd2646a1758d",
                       "fwd": 1303.7e6, "adj": 1337.4e6,
                       "profile": "profiles/step3d_yee3d_256_fp32.md"},
    # one launch = eight time steps of the grid
    "te2d_2048_fp32": {"sources": SRC_TE, "sha256_16": "3577d4f00a6f53a3",
                       "fwd": 40.7e6, "adj": 50.9e6,
                       "profile": "profiles/step_te_multi_te2d_2048_fp32.md"},
}


def sources_sha(paths):
    """First 16 hex digits of the SHA-256 of the files' bytes, concatenated in order."""
    import hashlib
    h = hashlib.sha256()
    for p in paths:
        with open(os.path.join(ROOT, p), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def measured_traffic(name):
    rec = MEASURED_TRAFFIC.get(name)
    if rec is None:
        return None, None
    # the counters were taken with the default schedules (2D: several steps
    # per launch; 3D: one)
    tb = os.environ.get("FDTD_TEMPORAL_BLOCKING", "")
    if (tb == "0" and rec["sources"] in (SRC_2D, SRC_BATCH, SRC_TE)) or (tb == "1" and rec["sources"] is SRC_3D):
        return None, None
    try:
        h = sources_sha(rec["sources"])
    except OSError:
        return None, None
    if h != rec["sha256_16"]:
        return None, None
    return rec, 0.5 * (rec["fwd"] + rec["adj"])


def algorithmic_bytes(w, adjoint):
    """HBM bytes one launch of the fused step kernel must move at minimum:
    every field array read once and written once; absorber memories over the
    CPML strips; density, Drude current and history (forward: write;
    adjoint: read, plus the FP64 sensitivity sum) over the design box."""
    esz = 4 if w["precision"] == 32 else 8
    nx, ny, nz = w["n"]
    P = w["pml_cells"]
    dnx, dny, dnz = w["design_n"]
    if w["dims"] == 2:
        cells = nx * ny
        fields = 3
        pml_cells = 2 * (2 * P) * (nx + ny)  # psi_E and psi_H per strip direction
        design = W.te_edges(w["design_n"])[1] if W.is_te(w) else dnx * dny  # TEz: one value per edge
        ncomp = 1
    else:
        cells = nx * ny * nz
        fields = 6
        pml_cells = 4 * (2 * P) * (ny * nz + nx * nz + nx * ny)
        design = dnx * dny * dnz
        ncomp = 3
    b = cells * fields * 2 * esz + pml_cells * 2 * esz
    if not adjoint:
        b += design * (esz + ncomp * (2 * esz + esz))            # rho; J r/w + history write
    else:
        b += design * (esz + ncomp * (2 * esz + esz + 16))       # rho; J r/w + history read + FP64 sum r/w
    return b


def cpu_baseline(w, steps):
    """The oracle as it stands, on the first `steps` steps of the workload."""
    import oracle
    ws = W.with_(w, n_steps=steps, precision=64)
    o = oracle.Oracle(ws)
    rho = W.seeded_rho(ws, 0)
    t0 = time.perf_counter()
    o.set_density(rho)
    o.forward()
    o.adjoint()
    o.gradient()
    dt = time.perf_counter() - t0
    nx, ny, nz = w["n"]
    cells = nx * ny * (nz if w["dims"] == 3 else 1)
    o.close()
    return {"value": cells * steps * 2 / dt / 1e9, "unit": "Gcell-updates/s", "cores": oracle.num_threads(),
            "kind": "oracle",
            "sample": f"{w['name']} grid, first {steps} of {w['n_steps']} steps, forward+adjoint+gradient, "
                      f"FP64, {dt:.1f} s wall"}


def bench_c4(args):
    """The batched uneven workload: 64 2D FP32 instances (sides 128-1024, own
    damping and band) advanced together by fdtd_batch_* with the batch-tuned
    tile and temporal-block depths and graph replay; one bench step = set
    every density, batched forward, batched adjoint, every gradient."""
    import torch
    import paper_2203_01462_amd as P

    ws = W.c4(n_steps=args.n_steps or 5000)
    stream = torch.cuda.Stream()
    t0 = time.perf_counter()
    b = P.Batch(ws, stream=stream.cuda_stream, rows=0, use_graph=True, depth=0)
    setup_s = time.perf_counter() - t0
    with torch.cuda.stream(stream):
        rhos = [torch.from_numpy(W.seeded_rho(w, k).astype(np.float32)).to("cuda") for k, w in enumerate(ws)]
        grads = [torch.empty_like(r) for r in rhos]
    stream.synchronize()

    def step():
        for k, r in enumerate(rhos):
            b.set_density(k, r)
        b.forward()
        b.adjoint()
        for k, g in enumerate(grads):
            b.gradient(k, g)

    for _ in range(args.warmup):
        step()
    stream.synchronize()
    torch.cuda.synchronize()
    fwd_ms = adj_ms = 0.0
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
        stream.synchronize()
        i = b.info(0)
        fwd_ms += i["forward_ms"]
        adj_ms += i["adjoint_ms"]
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    info = [b.info(k) for k in range(len(ws))]
    b.close()
    N = ws[0]["n_steps"]
    value = sum(W.cell_updates(w) for w in ws) / (wall / args.steps) / 1e9
    bf = sum(algorithmic_bytes(w, False) for w in ws)
    ba = sum(algorithmic_bytes(w, True) for w in ws)
    achieved = (bf + ba) * N * args.steps / ((fwd_ms + adj_ms) * 1e-3) / 1e9
    trec, traffic = measured_traffic("tmz2d_batch64_c4")
    depth_by_side = sorted({(w["n"][0], i["depth"]) for w, i in zip(ws, info)})
    out = {
        "metric": METRIC, "value": round(value, 3), "unit": "Gcell-updates/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(wall / args.steps * 1e3, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "tmz2d_batch64_c4", "instances": len(ws),
                   "sides": sorted({w["n"][0] for w in ws}), "time_steps": N, "n_freq": ws[0]["n_freq"],
                   "tile_depths": sorted({i["rows"] for i in info}),
                   "temporal_block_depth_by_side": [list(x) for x in depth_by_side],
                   "setup_and_tuning_s": round(setup_s, 2), "density": "seeded smoothed U[0,1), seed = index",
                   "parallelism": "single GPU"},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                     "traffic_per_step_fwd_adj": [trec["fwd"], trec["adj"]] if trec else None,
                     "kernel": "step2d_batch_mix_kernel (all instances, two launches per two time steps)",
                     "bytes_per_step_fwd": bf, "bytes_per_step_adj": ba,
                     "avg_step_us_fwd": round(fwd_ms * 1e3 / (N * args.steps), 3),
                     "avg_step_us_adj": round(adj_ms * 1e3 / (N * args.steps), 3)},
    }
    if not args.no_cpu:
        out["cpu_baseline"] = cpu_baseline_c4(ws, args.cpu_steps or 2000)
    print(json.dumps(out), flush=True)


def cpu_baseline_c4(ws, steps):
    """The oracle as it stands on one instance of each side of the batch,
    first `steps` steps each."""
    import oracle
    seen, cells_steps, dt = set(), 0, 0.0
    for k, w in enumerate(ws):
        side = w["n"][0]
        if side in seen:
            continue
        seen.add(side)
        ws1 = W.with_(w, n_steps=min(steps, w["n_steps"]), precision=64)
        o = oracle.Oracle(ws1)
        rho = W.seeded_rho(ws1, k)
        t0 = time.perf_counter()
        o.set_density(rho)
        o.forward()
        o.adjoint()
        o.gradient()
        dt += time.perf_counter() - t0
        o.close()
        cells_steps += W.cell_updates(ws1)
    return {"value": cells_steps / dt / 1e9, "unit": "Gcell-updates/s", "cores": oracle.num_threads(),
            "kind": "oracle",
            "sample": f"one instance of each side {sorted(seen)}, first {steps} steps each, forward+adjoint+"
                      f"gradient, FP64, {dt:.1f} s wall"}


MFMA_BF16_PEAK_TFLOPS = 2500.0


def bench_unet(args, batch=32, side=128, inner=20):
    """Training steps of the surrogate U-Net (forward, backward, Adam) on
    seeded synthetic 128x128 densities and targets; one bench step = `inner`
    training steps.  Roofline: the convolutions' FLOPs (forward, data and
    weight gradients: 3x the forward) over the wall time of the whole step,
    against the dense BF16 matrix-core peak."""
    import torch
    from paper_2203_01462_amd.nn import UNet, layer_plan

    torch.cuda.set_device(0)
    stream = torch.cuda.Stream()
    g = torch.Generator().manual_seed(0)
    with torch.cuda.stream(stream):
        net = UNet(side, batch, seed=0)
        rho = torch.rand(batch, side, side, generator=g).cuda()
        Ft = torch.randn(batch, generator=g).cuda()
        St = torch.randn(batch, side, side, generator=g).cuda()

        def step():
            for _ in range(inner):
                net.forward(rho)
                dF, dS = net.loss_grad(Ft, St)
                net.backward(dF, dS)
                net.step(1e-4)

        for _ in range(args.warmup):
            step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            step()
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
    per_train_step = wall / (args.steps * inner)
    fwd_flops = sum(2 * ci * 9 * co * (side >> lvl) ** 2 for ci, co, lvl in layer_plan()) * batch
    tflops = 3 * fwd_flops / per_train_step / 1e12
    out = {"metric": "surrogate U-Net training samples/s (BF16 matrix cores)", "value": round(batch / per_train_step, 1),
           "unit": "samples/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
           "ms_per_step": round(wall / args.steps * 1e3, 3), "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
           "config": {"workload": f"unet_{side}_b{batch}", "channels": [32, 64, 128, 256], "batch": batch,
                      "input": [side, side], "train_steps_per_step": inner, "parallelism": "single GPU"},
           "roofline": {"bound": "mfma", "achieved": round(tflops, 2), "peak": MFMA_BF16_PEAK_TFLOPS,
                        "unit": "TFLOP/s", "frac": round(tflops / MFMA_BF16_PEAK_TFLOPS, 4), "traffic": None,
                        "kernel": "whole training step (convolution FLOPs / step time)",
                        "ms_per_train_step": round(per_train_step * 1e3, 3)}}
    print(json.dumps(out), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="c3", choices=["c1", "c2", "c3", "c4", "te", "unet"],
                    help="c4: 64 uneven 2D instances batched; te: 2D TEz (E in the plane) at 2048^2; "
                         "unet: training steps of the surrogate network "
                         "(BF16 matrix cores) instead of FDTD")
    ap.add_argument("--n-steps", type=int, default=0, help="override the time steps of a solve (testing only)")
    ap.add_argument("--cpu-steps", type=int, default=0,
                    help="time steps of the oracle sample (0: 200 for the 3D grid, 2000 otherwise)")
    ap.add_argument("--ckpt-every", type=int, default=0,
                    help="checkpoint the forward every K steps (0: store the full history)")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--copy-probe", action="store_true",
                    help="only run 5 device copies of 1 GiB (calibrates HBM byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: the solver runs on a single device and is measured on one GPU only; "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2203_01462_amd as P

    torch.cuda.set_device(0)
    if args.copy_probe:
        src = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes_read_per_dispatch": src.numel() * 4,
                          "copy_probe_bytes_written_per_dispatch": dst.numel() * 4}), flush=True)
        return
    if args.workload == "unet":
        bench_unet(args)
        return
    if args.workload == "c4":
        bench_c4(args)
        return
    base = W.PRESETS[args.workload]()
    if args.n_steps:
        base = W.with_(base, n_steps=args.n_steps)
    gmults = [1.0, 4.0, 16.0] if args.workload == "c2" else [1.0]
    stream = torch.cuda.Stream()
    ctxs = [P.FDTD(W.with_(base, gamma_mult=g), stream=stream.cuda_stream, ckpt_every=args.ckpt_every)
            for g in gmults]
    dt_np = np.float32 if base["precision"] == 32 else np.float64
    rho_host = W.seeded_rho(base, 0).astype(dt_np)
    with torch.cuda.stream(stream):
        rho = torch.from_numpy(rho_host).to("cuda")
        grad = torch.empty_like(rho)
    stream.synchronize()

    def step(i):
        c = ctxs[i % len(ctxs)]
        c.set_density(rho)
        c.forward()
        c.adjoint()
        c.gradient(grad)
        return c

    for i in range(args.warmup):
        step(i)
    stream.synchronize()
    torch.cuda.synchronize()
    fwd_ms = adj_ms = 0.0
    launches_f = launches_a = 0
    t0 = time.perf_counter()
    for i in range(args.steps):
        c = step(args.warmup + i)
        stream.synchronize()
        t = c.timing()
        fwd_ms += t["forward_ms"]
        adj_ms += t["adjoint_ms"]
        launches_f += t["forward_launches"]
        launches_a += t["adjoint_launches"]
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms_per_step = wall / args.steps * 1e3
    cells_steps = W.cell_updates(base)  # cells x N x 2
    value = cells_steps / (wall / args.steps) / 1e9

    bf = algorithmic_bytes(base, False)
    ba = algorithmic_bytes(base, True)
    achieved = (bf * launches_f + ba * launches_a) / ((fwd_ms + adj_ms) * 1e-3) / 1e9
    trec, traffic = measured_traffic(base["name"])
    step_s = (fwd_ms + adj_ms) * 1e-3 / max(launches_f + launches_a, 1)
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                "achieved_is": "algorithmic bytes per time step / event time per step (effective bandwidth)",
                "traffic_per_step_fwd_adj": [trec["fwd"], trec["adj"]] if trec else None,
                # counter-measured HBM bytes per step over the same event time
                "measured_gbs": round(traffic / step_s / 1e9, 1) if traffic else None,
                "measured_frac": round(traffic / step_s / 1e9 / HBM_PEAK_GBS, 4) if traffic else None,
                "kernel": ("step_te_multi (several time steps per launch)" if W.is_te(base)
                           else "step2d_multi (several time steps per launch)" if base["dims"] == 2
                           else "step3d_general_fwd (forward) or step3d_general x3 (adjoint) + step3d_plain"
                                " (one time step)"),
                "bytes_per_step_fwd": bf, "bytes_per_step_adj": ba,
                "avg_step_us_fwd": round(fwd_ms * 1e3 / max(launches_f, 1), 3),
                "avg_step_us_adj": round(adj_ms * 1e3 / max(launches_a, 1), 3)}
    nx, ny, nz = base["n"]
    out = {
        "metric": METRIC, "value": round(value, 3), "unit": "Gcell-updates/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_per_step, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32" if base["precision"] == 32 else "f64", "data": "synthetic",
        "config": {"workload": base["name"], "grid": [nx, ny] if base["dims"] == 2 else [nx, ny, nz],
                   "dx_nm": base["dx"] * 1e9, "time_steps": base["n_steps"], "pml_cells": base["pml_cells"],
                   "design_box": list(base["design_n"][:base["dims"]]), "gap_box": list(base["gap_n"][:base["dims"]]),
                   "n_freq": base["n_freq"], "gamma_mult_cycle": gmults, "density": "seeded smoothed U[0,1), seed 0",
                   "ckpt_every": args.ckpt_every,
                   "parallelism": "single GPU"},
        "roofline": roofline,
    }
    for c in ctxs:
        c.close()
    if not args.no_cpu:
        cs = args.cpu_steps or (200 if base["dims"] == 3 else 1000 if W.is_te(base) else 2000)
        out["cpu_baseline"] = cpu_baseline(base, min(cs, base["n_steps"]))
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
