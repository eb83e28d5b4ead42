#!/usr/bin/env python3
"""Benchmark of the hot path: energy + gradient + SPD-projected block-CSR
Hessian of the elastic-shell objective (StVK membrane per triangle + dihedral
bending per interior-edge diamond), FP32 derivative arithmetic, FP64 energy.

Workloads:
  shell   (default) 1024 x 1024-vertex grid rolled into a half cylinder with
          N(0, (1e-3 h)^2) noise: 2,093,058 triangles, 3,137,541 diamonds,
          13,606,924 3x3 blocks.
  batched 700 geodesic icospheres of lognormal size (one mesh of disjoint
          components, per-component FP64 energies), layout chosen by the
          autotuner; also timed as one evaluation per mesh.
  mlp     the learned per-triangle density on a 708 x 708 shell.
  cloth   mass-spring cloth time step (Sec. 7.1): springs on the 2,996,001 edges
          of a 1000 x 1000 grid plus inertia and gravity per vertex, filtered
          Hessian; also timed at the Table 1 sizes 10^2 ... 1000^2 vertices.
  symdir  symmetric Dirichlet parameterisation energy (Sec. 7.2) on a 1001 x 1001
          disk-topology grid (2,000,000 triangles) with UVs warped by 8 seeded
          sinusoids: 2 DOFs per vertex, 2x2 blocks, eigen-clamped 6x6 element
          Hessians.

One step = one mad_problem_eval(ENERGY | GRAD | HESS | SPD) over the whole
workload with inputs resident in HBM (topology, patches and pattern are built
once, outside the timed region). Prints one JSON line.

  python bench.py [--gpus 1] [--steps 50] [--warmup 10] [--precision f32|f64]
                  [--workload shell|batched] [--n 1024] [--no-cpu-baseline]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# Executed floating-point operations per element of the fused patch kernel on the 1024^2 shell
# workload (FP32 + FP64 VALU wave instructions x 64 lanes, FMA = 2), and its HBM traffic per launch
# (FETCH_SIZE x 2.00 + WRITE_SIZE x 1.00, factors from a 1 GiB copy), from the rocprofv3 counter
# passes in profiles/k_eval_patch_f32_shell1024_counters.md. Valid for the kernel as profiled there.
FLOPS_PER_ELEM = {"f32": 9069.1, "f64": None}
# traffic at the default layout (444-face patches, 4 waves, the dispatcher as the queue)
TRAFFIC_BYTES = {"f32": 0.9806e9, "f64": None}
# the same for the 1000^2 cloth step, evaluated by rows (profiles/k_eval_rows_f32_cloth1000_counters.md)
CLOTH_TRAFFIC_BYTES = {"f32": 0.4545e9, "f64": None}
# and for the 1001^2 symmetric Dirichlet parameterisation at its default layout (512-face patches;
# profiles/k_eval_patch_f32_symdir1001_trace_counters.md)
SYMDIR_TRAFFIC_BYTES = {"f32": 0.3430e9, "f64": None}

# MI355X published peaks used as roofline denominators
HBM_PEAK_GBS = 8000.0
VALU_PEAK_TFLOPS = {"f32": 157.3, "f64": 78.6}
# the FP32 vector rate without packed FP32 instructions (this build disables them): half the published figure
VALU_UNPACKED_TFLOPS = {"f32": 78.6, "f64": 78.6}

SHELL_TERMS = ((4, (1.0, 1.0)), (5, (1.0, 1.0)))   # StVK (mu, lambda), bending (k_b, h)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--precision", choices=["f32", "f64"], default="f32")
    ap.add_argument("--workload", choices=["shell", "batched", "mlp", "cloth", "symdir"], default="shell")
    ap.add_argument("--symdir-n", type=int, default=1001, help="grid side of the parameterisation workload")
    ap.add_argument("--cloth-n", type=int, default=1000, help="grid side of the cloth workload")
    ap.add_argument("--n", type=int, default=1024, help="grid side of the shell workload")
    ap.add_argument("--meshes", type=int, default=700, help="meshes of the batched workload")
    ap.add_argument("--mlp-n", type=int, default=708, help="grid side of the learned-density workload")
    ap.add_argument("--patch-faces", type=int, default=0)
    ap.add_argument("--scatter", choices=["patch", "atomic", "color"], default="patch")
    ap.add_argument("--persistent", action="store_true", help="persistent launch (the default for heavy terms)")
    ap.add_argument("--per-patch", action="store_true", help="one workgroup per patch")
    ap.add_argument("--wg-waves", type=int, choices=[0, 4, 8], default=0,
                    help="patch kernel tile: waves per workgroup (0: the default 4)")
    ap.add_argument("--autotune", action="store_true", help="choose the layout by timing (batched: always)")
    ap.add_argument("--no-fp64-plain", action="store_true", help="skip the FP64 GPU comparison run")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-sizes", action="store_true",
                    help="cloth: skip the Table 1 size sweep; symdir: skip the Table 2 product sweep")
    ap.add_argument("--no-hvp", action="store_true", help="shell, symdir: skip the matrix-free product timing")
    ap.add_argument("--no-dynamic", action="store_true", help="shell: skip the pair-insertion timing")
    ap.add_argument("--no-jacobian", action="store_true", help="cloth: skip the residual Jacobian timing")
    ap.add_argument("--pairs", type=int, default=100000, help="interaction pairs inserted by the dynamic timing")
    ap.add_argument("--cpu-elements", type=int, default=300000, help="elements in the oracle timing sample")
    ap.add_argument("--summarize-counters", metavar="DIR", default=None,
                    help="summarise a rocprofv3 counter-collection CSV under DIR and exit")
    ap.add_argument("--copy-bytes", type=int, default=0,
                    help="run only a device-to-device copy of this many bytes (traffic-counter calibration)")
    return ap.parse_args()


def alg_bytes(nv, nt, nd, nnzb, precision_bytes):
    """Algorithmic HBM bytes of one step: x, triangles, diamonds, per-element rest data and the
    pattern read once; gradient, every Hessian value and the energy written once."""
    rd = nv * 3 * 8 + nt * 3 * 4 + nd * 4 * 4 + nt * 5 * 8 + nd * 2 * 8 + (nv + 1) * 4 + nnzb * 4
    wr = nv * 3 * precision_bytes + nnzb * 9 * precision_bytes + 8
    return rd + wr


def workload(args):
    from paper_2509_00406_amd import meshgen
    if args.workload == "shell":
        inp = meshgen.shell_cylinder(n=args.n, seed=2001)
        desc = (f"elastic shell StVK+bending, {args.n}x{args.n} grid half cylinder, noise sigma=1e-3 h, "
                f"SPD-projected Hessians, block-CSR 3x3")
    elif args.workload == "batched":
        inp = meshgen.icosphere_batch(n_meshes=args.meshes)
        desc = (f"batched: {args.meshes} geodesic icospheres (lognormal sizes), StVK+bending, one launch, "
                f"per-mesh FP64 energies, SPD-projected Hessians, block-CSR 3x3")
    elif args.workload == "symdir":
        inp = meshgen.warped_grid(n=args.symdir_n, seed=3001)
        desc = (f"symmetric Dirichlet parameterisation, {args.symdir_n}x{args.symdir_n} disk grid, UVs warped by 8 "
                f"seeded sinusoids (amplitude 0.1), 2 DOFs per vertex, SPD-projected Hessians, block-CSR 2x2")
    elif args.workload == "cloth":
        inp = meshgen.cloth(n=args.cloth_n, seed=6001)
        desc = (f"mass-spring cloth step: springs on every edge + inertia and gravity per vertex, "
                f"{args.cloth_n}x{args.cloth_n} grid, filtered (SPD-projected) Hessians, block-CSR 3x3")
    else:
        inp = meshgen.shell_cylinder(n=args.mlp_n, seed=5001)
        desc = (f"learned density: 6-64-64-1 softplus network per triangle (BF16 weights, FP32 accumulation on "
                f"MFMA), forward-mode grad + SPD-projected 9x9 Hessian, {args.mlp_n}x{args.mlp_n} grid half "
                f"cylinder, block-CSR 3x3")
    return inp, desc


def density_network(mad):
    """The trained shell density (paper_2509_00406_amd/data, written by tests/train_density.py), else a
    network with seeded random weights (evaluation speed does not depend on the values)."""
    if os.path.exists(mad.TRAINED_DENSITY):
        return mad.Network.from_file(mad.TRAINED_DENSITY), "trained"
    return seeded_network(mad), "seeded random weights (no trained parameters found)"


def seeded_network(mad, seed=5003):
    """A network with seeded random weights (evaluation speed does not depend on the values)."""
    import numpy as np
    r = np.random.default_rng(seed)
    H = mad.MLP_HIDDEN
    theta = np.concatenate([r.normal(scale=0.5, size=6 * H), r.normal(scale=0.5, size=H),
                            r.normal(scale=1.0 / H ** 0.5, size=H * H), r.normal(scale=0.5, size=H),
                            r.normal(scale=0.3, size=H), [0.1]]).astype(np.float32)
    return mad.Network(theta, np.array([60, 60, 80, 2, 1, 2], np.float32), 1.0)


def cpu_sample(inp, budget, per_vertex=5.0):
    """A bounded piece of the workload for the oracle: leading grid rows of the shell, or the first
    meshes of the batch, about `budget` elements (`per_vertex` elements per vertex)."""
    import numpy as np
    if inp.comp_offsets is None:
        n = inp.meta["n"]
        rows = max(2, min(n, int(budget / (per_vertex * n))))
        nv = rows * n
        what = f"first {rows} of {n} grid rows of the same shell"
    else:
        co = inp.comp_offsets
        k, nv = 0, 0
        while k < len(co) - 1 and (k == 0 or 5.0 * (co[k + 1] - 0) <= budget):
            k += 1
        nv = int(co[k])
        what = f"first {k} of {len(co) - 1} meshes of the same batch"
    sel = np.all(inp.tris < nv, axis=1)
    return inp.tris[sel], inp.rest[:nv], inp.x[:nv], nv, what


def cpu_baseline(inp, budget, mlp=None):
    """The FP64 oracle timed on a bounded sample of the same workload (serial C). With a network:
    the learned-density form (the oracle gets the same parameters in FP64)."""
    import numpy as np
    from oracle import oracle as O
    tris, rest, x, nv, what = cpu_sample(inp, budget, per_vertex=2.0 if mlp is not None else 5.0)
    P = O.Problem(tris, rest, nv, 3)
    if mlp is not None:
        t = mlp.params(1).astype(np.float64)
        H = 64
        W1, b1 = t[:6 * H].reshape(H, 6), t[6 * H:7 * H]
        W2, b2 = t[7 * H:7 * H + H * H].reshape(H, H), t[7 * H + H * H:8 * H + H * H]
        w3, b3 = t[8 * H + H * H:9 * H + H * H], t[9 * H + H * H]
        P.add_term(O.MLP, O.mlp_pack(mlp.s_out, mlp.s_in.astype(np.float64), W1, b1, W2, b2, w3, b3))
    else:
        for k, prm in SHELL_TERMS:
            P.add_term({4: O.STVK, 5: O.BENDING}[k], prm)
    P.build_pattern()
    n_el = int(tris.shape[0]) + (int(P.topo.diamonds.shape[0]) if mlp is None else 0)
    kind = "learned-density triangles" if mlp is not None else "StVK triangles + bending diamonds"
    return time_oracle(P, x, n_el, f"{what}: {n_el} elements ({kind}), energy + gradient + SPD-projected Hessian "
                                   f"+ assembly, FP64")


def host_threads():
    """Threads the oracle may use here: this process's CPU affinity, capped by OMP_NUM_THREADS if set."""
    n = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else (os.cpu_count() or 1)
    env = os.environ.get("OMP_NUM_THREADS", "")
    if env.isdigit() and int(env) > 0:
        n = min(n, int(env))
    return max(1, n)


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def time_oracle(P, x, n_el, what):
    """The FP64 oracle on one sample, four ways: its parity build (gcc -O2, no FMA contraction) on all the
    host threads this process may use (the reported value) and on one thread, and its -O3 -march=native
    timing build on one and on all threads. The threaded evaluation is bit-identical to the serial one
    (per-element work in parallel, each block row summed by one thread in the serial order)."""
    from oracle import oracle as O
    mode = O.ENERGY | O.GRAD | O.HESS | O.SPD
    nth = host_threads()

    def timed(fn):
        t0 = time.perf_counter()
        fn()
        return time.perf_counter() - t0
    t1 = timed(lambda: P.eval(x, mode, scales=False))
    tn = timed(lambda: P.eval_par(x, mode, threads=nth))
    fast = {}
    try:
        with O.using(O.load(O.build_fast())):
            f1 = timed(lambda: P.eval_par(x, mode, threads=1))
            fn_ = timed(lambda: P.eval_par(x, mode, threads=nth))
        fast = {"one_thread": n_el / f1, "all_threads": n_el / fn_, "build": "gcc -O3 -march=native -fopenmp"}
    except Exception as exc:   # a host without a working gcc: report the parity build only
        fast = {"error": str(exc)[:200]}
    return {"value": n_el / tn, "unit": "elements/s", "cores": nth, "kind": "oracle",
            "sample": f"{what}; parity build (gcc -O2 -ffp-contract=off), {nth} threads, {tn:.2f} s "
                      f"(one thread {t1:.1f} s) on {cpu_model()}; host nproc {os.cpu_count()}",
            "one_thread": n_el / t1, "o3_native": fast}


def summarize_counters(path, n_elements):
    """Per-dispatch averages of every counter of every kernel in a rocprofv3 counter CSV, plus the
    FP operation count of the FP32/FP64 VALU counters (each wave instruction counted as 64 lanes,
    FMA as 2 operations) per element of the shell workload."""
    import csv
    import glob
    from collections import defaultdict
    files = glob.glob(os.path.join(path, "**", "*counter_collection.csv"), recursive=True)
    out = {}
    for f in files:
        agg = defaultdict(lambda: defaultdict(float))
        disp = defaultdict(set)
        for r in csv.DictReader(open(f)):
            agg[r["Kernel_Name"]][r["Counter_Name"]] += float(r["Counter_Value"])
            disp[r["Kernel_Name"]].add(r["Dispatch_Id"])
        for k, d in agg.items():
            n = len(disp[k])
            e = out.setdefault(k, {"dispatches": n})
            e.update({c: v / n for c, v in d.items()})
    for k, e in out.items():
        ops = 0.0
        for prec in ("F32", "F64"):
            ops += 2 * e.get(f"SQ_INSTS_VALU_FMA_{prec}", 0.0) + e.get(f"SQ_INSTS_VALU_ADD_{prec}", 0.0) + \
                   e.get(f"SQ_INSTS_VALU_MUL_{prec}", 0.0) + e.get(f"SQ_INSTS_VALU_TRANS_{prec}", 0.0)
        if ops:
            e["fp_ops_per_dispatch"] = 64 * ops
            e["fp_ops_per_element"] = 64 * ops / n_elements
    return out


def copy_calibration(nbytes):
    import torch
    src = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda").fill_(1.0)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes": nbytes, "note": "each copy reads and writes this many bytes"}), flush=True)


def copy_bandwidth(nbytes=1 << 30, reps=5):
    """Device-to-device copy rate (bytes read + written per second, GB/s): the reachable HBM
    rate this box shows for a plain stream, beside the published 8 TB/s."""
    import torch
    src = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda").fill_(1.0)
    dst = torch.empty_like(src)
    dst.copy_(src)
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0.record()
    for _ in range(reps):
        dst.copy_(src)
    t1.record()
    torch.cuda.synchronize()
    gbs = 2 * nbytes * reps / (t0.elapsed_time(t1) * 1e-3) / 1e9
    del src, dst
    torch.cuda.empty_cache()
    return gbs


def make_problem(mad, mesh, inp, prec, args, stream, form=None):
    """form: "plain" (StVK + bending), "mlp" (learned density), "analytic" (shell-triangle density),
    "cloth" (springs + inertia); default: the workload's own."""
    form = form or {"mlp": "mlp", "cloth": "cloth", "symdir": "symdir"}.get(args.workload, "plain")
    scatter = {"patch": mad.SCATTER_PATCH, "atomic": mad.SCATTER_ATOMIC, "color": mad.SCATTER_COLOR}[args.scatter]
    prob = mad.Problem(mesh, 2 if form == "symdir" else 3, prec, patch_faces=args.patch_faces, scatter=scatter,
                       wg_waves=args.wg_waves)
    if form == "symdir":
        prob.add_term(mad.SYMDIR, (), inp.rest)
    elif form == "cloth":
        import torch
        prob.add_term(mad.SPRING, inp.meta["spring_params"], inp.rest)
        prob.add_vertex_term(mad.INERTIA, inp.meta["inertia_params"], torch.from_numpy(inp.meta["vdata"]).cuda())
    elif form == "mlp":
        prob.add_mlp_term(density_network(mad)[0], inp.rest)
    elif form == "analytic":
        prob.add_term(mad.SHELL_TRI, (1.0, 1.0, 1.0), inp.rest)
    else:
        for k, prm in SHELL_TERMS:
            prob.add_term(k, prm, inp.rest)
    prob.finalize(stream)
    if args.persistent or args.per_patch:
        lay = prob.layout()
        prob.set_layout(lay["scatter"], lay["patch_faces"], 1 if args.persistent else 0, stream=stream)
    return prob


def time_steps(torch, fn, steps, warmup, stream):
    """Per-step HIP event times (ms) of `steps` calls after `warmup` untimed ones, and the
    wall-clock total of the timed region."""
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    t0 = time.perf_counter()
    evs[0].record(stream)
    for i in range(steps):
        fn()
        evs[i + 1].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    return [evs[i].elapsed_time(evs[i + 1]) for i in range(steps)], wall


def pct(v, q):
    import numpy as np
    return float(np.percentile(np.asarray(v), q))


def main():
    args = parse()
    if args.summarize_counters:
        print(json.dumps(summarize_counters(args.summarize_counters, 5230599), indent=1))
        return
    if args.copy_bytes:
        copy_calibration(args.copy_bytes)
        return
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU only; --gpus must be 1",
                          "n_gpus": args.gpus}), flush=True)
        sys.exit(2)
    import numpy as np
    import torch

    from paper_2509_00406_amd import mad

    assert torch.cuda.is_available(), "bench needs a GPU"
    torch.cuda.set_device(0)
    prec = mad.F32 if args.precision == "f32" else mad.F64
    pb = 4 if prec == mad.F32 else 8
    inp, desc = workload(args)
    stream = torch.cuda.current_stream()
    t0 = time.perf_counter()
    mesh = mad.Mesh(inp.tris, inp.n_verts, inp.comp_offsets)
    prob = make_problem(mad, mesh, inp, prec, args, stream)
    torch.cuda.synchronize()
    setup_s = time.perf_counter() - t0
    x = torch.from_numpy(inp.x.ravel().copy()).cuda()
    out = prob.outputs()
    mode = mad.ENERGY | mad.GRAD | mad.HESS | mad.SPD
    if args.workload == "cloth":
        n_elem = mesh.n_edges + mesh.n_verts
    elif args.workload == "symdir":
        n_elem = mesh.n_tris
    else:
        n_elem = mesh.n_tris + (mesh.n_diamonds if args.workload != "mlp" else 0)
    tune = None
    if args.autotune or args.workload == "batched":
        t1 = time.perf_counter()
        tune = prob.autotune(x, mode, out=out, reps=5, force=True, stream=stream)
        tune["tune_s"] = time.perf_counter() - t1
    layout = prob.layout()

    step = lambda: prob.eval(x, mode, out=out, stream=stream)   # noqa: E731
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    # the timed steps run without stage events (each event adds a few microseconds to the step); a second pass
    # of as many steps records the stages, whose fused-kernel time is the roofline's
    step_ms, wall = time_steps(torch, step, args.steps, 0, stream)
    ms_per_step = max(wall * 1e3, sum(step_ms)) / args.steps
    mad.mad_problem_set_profiling(prob.handle, True)
    time_steps(torch, step, args.steps, 0, stream)
    mad.mad_problem_set_profiling(prob.handle, False)
    stage_ms, n_evals = mad.mad_problem_profile(prob.handle)
    nonfinite, fallbacks = prob.status()
    copy_gbs = copy_bandwidth()   # after the timed region

    n_terms = {"mlp": 1, "cloth": 2, "symdir": 1}.get(args.workload, len(SHELL_TERMS))
    if layout["scatter"] == mad.SCATTER_PATCH:
        dom_name = {"mlp": "k_eval_patch (learned-density chain + clamp + assembly)",
                    "cloth": "k_eval_rows (springs + inertia by rows)",
                    "symdir": "k_eval_patch (symmetric Dirichlet, 2x2 blocks)"}.get(args.workload,
                                                                          "k_eval_patch (StVK + bending fused)")
        dom_ms = stage_ms[2] / n_evals
        stages = {"fill": stage_ms[0] / n_evals, "network": stage_ms[1] / n_evals, "fused": stage_ms[2] / n_evals,
                  "gather_and_fp64_redo": stage_ms[3] / n_evals, "energy": stage_ms[-1] / n_evals}
    else:
        term_ms = stage_ms[2:2 + n_terms]
        dom = int(np.argmax(term_ms))
        dom_ms = term_ms[dom] / n_evals
        names = (["k_eval<spring>", "k_eval<inertia>"] if args.workload == "cloth"
                 else ["k_eval<symdir>"] if args.workload == "symdir"
                 else ["k_eval<StVK>", "k_eval<bending>"][:n_terms])
        dom_name = names[dom]
        stages = {"fill": stage_ms[0] / n_evals, **{nm: t / n_evals for nm, t in zip(names, term_ms)},
                  "energy": stage_ms[-1] / n_evals}
    if args.workload == "cloth":
        step_bytes = cloth_alg_bytes(mesh.n_verts, mesh.n_edges, prob.nnzb, pb)
    elif args.workload == "symdir":
        step_bytes = symdir_alg_bytes(mesh.n_verts, mesh.n_tris, prob.nnzb, pb)
    elif args.workload == "mlp":   # triangles only, 8 rest doubles each
        step_bytes = alg_bytes(mesh.n_verts, mesh.n_tris, 0, prob.nnzb, pb) + mesh.n_tris * 24
    else:
        step_bytes = alg_bytes(mesh.n_verts, mesh.n_tris, mesh.n_diamonds, prob.nnzb, pb)
    default_shell = args.workload == "shell" and args.n == 1024 and layout["scatter"] == mad.SCATTER_PATCH
    fpe = FLOPS_PER_ELEM.get(args.precision) if default_shell else None
    peak = VALU_PEAK_TFLOPS[args.precision]
    if args.workload == "symdir":
        # a 4x4 reduced Hessian per triangle: few operations per byte, so the HBM stream is the roofline
        achieved = step_bytes / (dom_ms * 1e-3) / 1e9
        at_1001 = (args.symdir_n == 1001 and layout["scatter"] == mad.SCATTER_PATCH and layout["patch_faces"] == 512
                   and layout["persistent"] != 2 and layout["wg_waves"] == 4)
        roofline = {"bound": "hbm", "kernel": dom_name, "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": achieved / HBM_PEAK_GBS,
                    "traffic": SYMDIR_TRAFFIC_BYTES.get(args.precision) if at_1001 else None, "kernel_ms": dom_ms,
                    "alg_bytes_per_launch": step_bytes}
    elif args.workload == "cloth":
        # springs are cheap (a scalar function of the length each): the row kernel is held to its HBM stream
        achieved = step_bytes / (dom_ms * 1e-3) / 1e9
        at_1000 = (args.cloth_n == 1000 and layout["scatter"] == mad.SCATTER_PATCH)   # by rows
        roofline = {"bound": "hbm", "kernel": dom_name, "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": achieved / HBM_PEAK_GBS,
                    "traffic": CLOTH_TRAFFIC_BYTES.get(args.precision) if at_1000 else None, "kernel_ms": dom_ms,
                    "alg_bytes_per_launch": step_bytes}
    elif fpe:
        achieved = fpe * n_elem / (dom_ms * 1e-3) / 1e12
        roofline = {"bound": "alu", "kernel": dom_name, "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                    "frac": achieved / peak,
                    "traffic": (TRAFFIC_BYTES.get(args.precision)
                                if layout["patch_faces"] == 444 and layout["persistent"] != 2 else None),
                    "kernel_ms": dom_ms,
                    "flops_per_element": fpe,
                    "frac_of_unpacked_fp32": achieved / VALU_UNPACKED_TFLOPS[args.precision],
                    "hbm_frac_alg": step_bytes / (dom_ms * 1e-3) / 1e9 / HBM_PEAK_GBS}
    else:
        roofline = {"bound": "alu", "kernel": dom_name, "achieved": None, "peak": peak, "unit": "TFLOP/s",
                    "frac": None, "traffic": None, "kernel_ms": dom_ms, "flops_per_element": None}

    res = {
        "metric": "elements/s for energy+grad+sparse Hessian assembly",
        "value": n_elem / (ms_per_step * 1e-3),
        "unit": "elements/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "step_ms_p10_p50_p90": [pct(step_ms, 10), pct(step_ms, 50), pct(step_ms, 90)],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.precision,
        "data": "synthetic",
        "config": {"workload": desc, **({"springs": mesh.n_edges} if args.workload == "cloth" else
                                        {"triangles": mesh.n_tris} if args.workload == "symdir" else
                                        {"triangles": mesh.n_tris, "diamonds": mesh.n_diamonds}),
                   "elements": n_elem, "vertices": mesh.n_verts, "nnzb": prob.nnzb, "precision": args.precision,
                   "layout": layout},
        "roofline": roofline,
        "hbm": {"alg_bytes_per_step": step_bytes, "alg_GBs": step_bytes / (ms_per_step * 1e-3) / 1e9,
                "frac_of_peak": step_bytes / (ms_per_step * 1e-3) / 1e9 / HBM_PEAK_GBS,
                "copy_GBs": copy_gbs, "frac_of_copy": step_bytes / (ms_per_step * 1e-3) / 1e9 / copy_gbs},
        "stages_ms_per_step": stages,
        "setup_s": setup_s,
        "fp64_fallbacks": fallbacks,
        "nonfinite": nonfinite,
    }
    if tune is not None:
        res["autotune"] = tune
    if args.workload == "mlp":
        # network pass (normals, features, MFMA contractions): algorithmic flops per triangle = 8 contractions
        # over the 64 hidden units (7 forward channels and u = W2^T v) x 64 x 2, plus the layer-1 second
        # derivatives (21 packed pairs x 64 units x 2); the matrix cores execute three BF16 passes of each of
        # the 8 (hi/mid/lo activations) and five of the last (three-term by two-term operands)
        net_ms = stage_ms[1] / n_evals
        per_tri = 8 * 64 * 64 * 2 + 21 * 64 * 2
        useful = per_tri * mesh.n_tris
        executed = (3 * 8 * 64 * 64 * 2 + 5 * 32 * 64 * 2) * mesh.n_tris
        res["network_pass"] = {"ms": net_ms, "useful_flops_per_triangle": per_tri,
                               "useful_TFLOPs": useful / (net_ms * 1e-3) / 1e12,
                               "mfma_bf16_peak": 2500.0,
                               "mfma_frac": useful / (net_ms * 1e-3) / 1e12 / 2500.0,
                               "executed_bf16_TFLOPs": executed / (net_ms * 1e-3) / 1e12,
                               "note": "mfma_frac counts the algorithmic contractions once; the matrix cores run "
                                       "them three or five times (BF16 terms of the FP32 operands)"}
        res["network"] = density_network(mad)[1]
        res["vs_other_forms"] = other_forms(torch, mad, mesh, inp, args, stream, x, ms_per_step)
        res["learned_vs_analytic"] = learned_vs_analytic(torch, mad, mesh, inp, args, stream, x, out)
    if args.workload in ("shell", "symdir") and not args.no_hvp:
        # the matrix-free mode: y = H v with each element's clamped Hessian applied in LDS, no assembly
        v = torch.randn_like(x)
        y = torch.empty_like(out[1])
        hmode = mad.SPD

        def prod():
            mad.mad_problem_hvp(prob.handle, x, v, hmode, None, None, y, stream)
        hv_ms, hv_wall = time_steps(torch, prod, max(10, args.steps // 2), 3, stream)
        hv = max(hv_wall * 1e3, sum(hv_ms)) / len(hv_ms)
        res["hvp"] = {"ms_per_product": hv, "elements_per_s": n_elem / (hv * 1e-3),
                      "note": "clamped Hessian-vector product, matrix-free (no assembly)"}
    if args.workload == "shell" and not args.no_dynamic:
        res["dynamic_sparsity"] = dynamic_sparsity(torch, mad, mesh, inp, prec, args, stream, x)
    if args.workload == "batched":
        res["one_launch_per_mesh"] = per_mesh_baseline(torch, mad, inp, prec, stream, ms_per_step, args)
    if args.workload == "cloth" and not args.no_sizes:
        res["table1_sizes"] = cloth_sizes(torch, mad, args, stream)
    if args.workload == "symdir" and not args.no_sizes and not args.no_hvp:
        res["table2_sizes"] = symdir_hvp_sizes(torch, mad, args, stream)
    if args.workload == "cloth" and not args.no_jacobian:
        res["residual_jacobian"] = residual_jacobian(torch, mad, args, prec, stream)
    if prec == mad.F32 and not args.no_fp64_plain:
        res["vs_fp64_plain"] = fp64_plain(torch, mad, mesh, inp, args, stream, x, out, ms_per_step)
    if not args.no_cpu_baseline:
        if args.workload == "mlp":
            res["cpu_baseline"] = cpu_baseline(inp, 7000, mlp=density_network(mad)[0])
        elif args.workload == "cloth":
            res["cpu_baseline"] = cpu_baseline_cloth(inp, 3 * args.cpu_elements)
        elif args.workload == "symdir":
            res["cpu_baseline"] = cpu_baseline_symdir(inp, 3 * args.cpu_elements)
        else:
            res["cpu_baseline"] = cpu_baseline(inp, args.cpu_elements)
    print(json.dumps(res), flush=True)


def cloth_alg_bytes(nv, ne, nnzb, precision_bytes):
    """Algorithmic HBM bytes of one cloth step: x, per-vertex (m, xhat), edges, spring rest data
    (l^2, 1/l^2) and the pattern read once; gradient, every Hessian value and the energy written once."""
    rd = nv * 3 * 8 + nv * 4 * 8 + ne * 2 * 4 + ne * 2 * 8 + (nv + 1) * 4 + nnzb * 4
    wr = nv * 3 * precision_bytes + nnzb * 9 * precision_bytes + 8
    return rd + wr


def symdir_alg_bytes(nv, nt, nnzb, precision_bytes):
    """Algorithmic HBM bytes of one parameterisation step: UVs (2 doubles per vertex), triangles, rest data
    (Dm^-1 and area: 5 doubles per triangle) and the pattern read once; gradient, every 2x2 Hessian block and
    the energy written once."""
    rd = nv * 2 * 8 + nt * 3 * 4 + nt * 5 * 8 + (nv + 1) * 4 + nnzb * 4
    wr = nv * 2 * precision_bytes + nnzb * 4 * precision_bytes + 8
    return rd + wr


def cpu_baseline_symdir(inp, budget):
    """The FP64 oracle on the leading grid rows of the same warped grid (serial C)."""
    import numpy as np
    from oracle import oracle as O
    n = inp.meta["n"]
    rows = max(2, min(n, int(budget / (2.0 * n))))
    nv = rows * n
    sel = np.all(inp.tris < nv, axis=1)
    P = O.Problem(inp.tris[sel], inp.rest[:nv], nv, 2)
    P.add_term(O.SYMDIR, ())
    P.build_pattern()
    n_el = int(sel.sum())
    return time_oracle(P, inp.x[:nv], n_el, f"first {rows} of {n} grid rows of the same warped grid: {n_el} "
                                            f"triangles, energy + gradient + SPD-projected Hessian + assembly, FP64")


# Table 1 of the paper (RTX 4090, precision not stated): grad + Hessian ms per step by vertex count
PAPER_TABLE1_MS = {10: 0.18, 50: 0.22, 100: 0.25, 500: 3.09, 1000: 11.7}


def residual_jacobian(torch, mad, args, prec, stream):
    """Residual terms and their sparse Jacobian (Eq. 3) on the cloth's grid: an edge-length residual on every
    edge and a positional residual on every vertex (a quarter of them pulled toward targets, weight 0
    elsewhere). Timed: the Jacobian (residuals r in FP64 and the row-owned CSR values J) and the Gauss-Newton
    evaluation through the patch assembly (energy 1/2 |r|^2, gradient J^T r, Hessian J^T J)."""
    import numpy as np
    from paper_2509_00406_amd import meshgen
    n = args.cloth_n
    tris, rest = meshgen.grid(n)
    rng = np.random.default_rng(7001)
    x = rest + 0.05 * rng.normal(size=rest.shape)
    vd = np.zeros((n * n, 4))
    vd[:, 0] = rng.uniform(0.5, 2.0, n * n) * (rng.random(n * n) < 0.25)
    vd[:, 1:] = rest + np.array([0.0, 0.0, 0.2]) + 0.05 * rng.normal(size=rest.shape)
    mesh = mad.Mesh(tris, n * n)
    prob = mad.Problem(mesh, 3, prec)
    prob.add_term(mad.RES_EDGE, (3.0,), rest)
    vdt = torch.from_numpy(np.ascontiguousarray(vd)).cuda()
    prob.add_vertex_term(mad.RES_POSITION, (), vdt)
    prob.finalize(stream)
    xt = torch.from_numpy(x.ravel().copy()).cuda()
    m, nnz = mad.mad_problem_jacobian_info(prob.handle)
    pb = 4 if prec == mad.F32 else 8
    r = torch.empty(m, dtype=torch.float64, device="cuda")
    vals = torch.empty(max(nnz, 1), dtype=torch.float32 if prec == mad.F32 else torch.float64, device="cuda")
    jac = lambda: mad.mad_problem_jacobian(prob.handle, xt, r, vals, stream)   # noqa: E731
    jac_ms, _ = time_steps(torch, jac, 20, 3, stream)
    out = prob.outputs()
    gn = lambda: prob.eval(xt, mad.ENERGY | mad.GRAD | mad.HESS, out=out, stream=stream)   # noqa: E731
    gn_ms, _ = time_steps(torch, gn, 20, 3, stream)
    jms = float(np.median(jac_ms))
    # algorithmic bytes of the Jacobian: x, edges, edge rest lengths and per-vertex (w, x_t) read once; r and the
    # values written once (the row pointers and columns are fixed at setup)
    ne, nv = mesh.n_edges, mesh.n_verts
    jbytes = nv * 3 * 8 + ne * 2 * 4 + ne * 8 + nv * 4 * 8 + m * 8 + nnz * pb
    return {"rows": m, "nnz": nnz, "edges": ne, "vertices": nv,
            "ms_jacobian": jms, "alg_bytes": jbytes, "jacobian_GBs": jbytes / (jms * 1e-3) / 1e9,
            "jacobian_hbm_frac": jbytes / (jms * 1e-3) / 1e9 / HBM_PEAK_GBS,
            "ms_gauss_newton_eval": float(np.median(gn_ms)),
            "gauss_newton_elements_per_s": (ne + nv) / (float(np.median(gn_ms)) * 1e-3),
            "note": "edge-length residuals on every edge + positional residuals on every vertex; the Gauss-Newton "
                    "evaluation assembles J^T r and J^T J through the row kernel"}


def cloth_sizes(torch, mad, args, stream):
    """The cloth step at the Table 1 sizes (FP32 and FP64), with the paper's numbers as context."""
    from paper_2509_00406_amd import meshgen
    mode = mad.ENERGY | mad.GRAD | mad.HESS | mad.SPD
    rows = []
    for n in sorted(PAPER_TABLE1_MS):
        inp = meshgen.cloth(n=n, seed=6001)
        mesh = mad.Mesh(inp.tris, inp.n_verts)
        x = torch.from_numpy(inp.x.ravel().copy()).cuda()
        row = {"vertices": n * n, "springs": mesh.n_edges, "paper_rtx4090_ms": PAPER_TABLE1_MS[n]}
        for prec, name in ((mad.F32, "f32"), (mad.F64, "f64")):
            p = make_problem(mad, mesh, inp, prec, args, stream, form="cloth")
            o = p.outputs()
            step_ms, wall = time_steps(torch, lambda: p.eval(x, mode, out=o, stream=stream), 20, 3, stream)
            row[f"ms_{name}"] = max(wall * 1e3, sum(step_ms)) / len(step_ms)
            del p, o
        rows.append(row)
    return rows


# Sec. 7.2, Table 2: time per conjugate-gradient iteration of the paper's matrix-free Newton solver
# (one Hessian-vector product plus the iteration's vector operations) for the symmetric Dirichlet
# energy, by vertex count, on an RTX 4090 (context, not a target)
PAPER_TABLE2_MS = {1550: 0.026, 160000: 0.108, 560000: 0.383, 1520000: 0.817, 1830000: 1.102}


def symdir_hvp_sizes(torch, mad, args, stream):
    """Matrix-free Hessian-vector products of the symmetric Dirichlet energy (FP32 and FP64, clamped and
    plain) on warped grids whose vertex counts are closest to the Table 2 rows."""
    from paper_2509_00406_amd import meshgen
    rows = []
    for nv in sorted(PAPER_TABLE2_MS):
        n = int(round(nv ** 0.5))
        inp = meshgen.warped_grid(n=n, seed=3001)
        mesh = mad.Mesh(inp.tris, inp.n_verts)
        x = torch.from_numpy(inp.x.ravel().copy()).cuda()
        v = torch.randn_like(x)
        row = {"vertices": n * n, "triangles": mesh.n_tris, "paper_rtx4090_ms_per_cg_iteration": PAPER_TABLE2_MS[nv]}
        for prec, name in ((mad.F32, "f32"), (mad.F64, "f64")):
            p = make_problem(mad, mesh, inp, prec, args, stream, form="symdir")
            y = torch.empty(x.numel(), dtype=torch.float32 if prec == mad.F32 else torch.float64, device=x.device)
            for hmode, tag in ((mad.SPD, "spd"), (0, "plain")):
                def prod():
                    mad.mad_problem_hvp(p.handle, x, v, hmode, None, None, y, stream)
                ms, wall = time_steps(torch, prod, 20, 3, stream)
                row[f"ms_{name}_{tag}"] = max(wall * 1e3, sum(ms)) / len(ms)
            del p, y
        rows.append(row)
    return rows


def cpu_baseline_cloth(inp, budget):
    """The FP64 oracle on the leading grid rows of the same cloth (serial C)."""
    import numpy as np
    from oracle import oracle as O
    n = inp.meta["n"]
    rows = max(2, min(n, int(budget / (4.0 * n))))
    nv = rows * n
    sel = np.all(inp.tris < nv, axis=1)
    P = O.Problem(inp.tris[sel], inp.rest[:nv], nv, 3)
    P.add_term(O.SPRING, inp.meta["spring_params"])
    P.add_term(O.INERTIA, inp.meta["inertia_params"], vertex_data=inp.meta["vdata"][:nv])
    P.build_pattern()
    n_el = int(P.topo.edges.shape[0]) + nv
    return time_oracle(P, inp.x[:nv], n_el, f"first {rows} of {n} grid rows of the same cloth: {n_el} elements "
                                            f"(springs + vertices), energy + gradient + filtered Hessian + assembly, "
                                            f"FP64")


def dynamic_sparsity(torch, mad, mesh, inp, prec, args, stream, x):
    """Sec. 6.3: insert random interaction pairs into the pattern of a fresh problem (GPU update into the
    second pattern buffer, wall clock including its final synchronisation), then time evaluations on the
    grown pattern."""
    import numpy as np
    p = mad.Problem(mesh, 3, prec, patch_faces=args.patch_faces)
    for k, prm in SHELL_TERMS:
        p.add_term(k, prm, inp.rest)
    p.reserve_pairs(args.pairs)
    p.finalize(stream)
    nnzb0 = p.nnzb
    pairs = torch.from_numpy(np.ascontiguousarray(
        np.random.default_rng(7001).integers(0, mesh.n_verts, size=(args.pairs, 2)), dtype=np.int32)).cuda()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    added = p.insert_pairs(pairs, stream)
    ms_insert = (time.perf_counter() - t0) * 1e3
    o = p.outputs()
    mode = mad.ENERGY | mad.GRAD | mad.HESS | mad.SPD
    step_ms, wall = time_steps(torch, lambda: p.eval(x, mode, out=o, stream=stream), max(5, args.steps // 5), 2,
                               stream)
    res = {"pairs": args.pairs, "blocks_before": nnzb0, "blocks_added": added, "ms_insert": ms_insert,
           "ms_per_step_after": max(wall * 1e3, sum(step_ms)) / len(step_ms)}
    del p, o
    return res


def other_forms(torch, mad, mesh, inp, args, stream, x, ms_mlp):
    """The same mesh with the plain StVK + dihedral form and with the analytic shell-triangle density."""
    out = {}
    mode = mad.ENERGY | mad.GRAD | mad.HESS | mad.SPD
    for form in ("plain", "analytic"):
        p = make_problem(mad, mesh, inp, mad.F32, args, stream, form=form)
        o = p.outputs()
        step_ms, wall = time_steps(torch, lambda: p.eval(x, mode, out=o, stream=stream), max(5, args.steps // 2),
                                   3, stream)
        ms = max(wall * 1e3, sum(step_ms)) / len(step_ms)
        n_el = mesh.n_tris + (mesh.n_diamonds if form == "plain" else 0)
        out[form] = {"ms_per_step": ms, "elements": n_el, "nnzb": p.nnzb,
                     "learned_speedup": ms / ms_mlp}
        del p, o
    return out


def learned_vs_analytic(torch, mad, mesh, inp, args, stream, x, out_mlp):
    """Relative errors (norm-wise, assembled outputs) of the timed learned term against the analytic density it
    was trained on, evaluated on the GPU on the same mesh (the benchmark's last evaluation is out_mlp)."""
    p = make_problem(mad, mesh, inp, mad.F32, args, stream, form="analytic")
    ea, ga, ha = p.eval(x, mad.ENERGY | mad.GRAD | mad.HESS | mad.SPD, stream=stream)
    torch.cuda.synchronize()
    em, gm, hm = out_mlp
    return {"energy": abs(float(em[0] - ea[0])) / abs(float(ea[0])), "grad": float((gm - ga).norm() / ga.norm()),
            "hess_clamped": float((hm - ha).norm() / ha.norm())}


def fp64_plain(torch, mad, mesh, inp, args, stream, x, out32, ms32):
    """The same evaluation on the FP64 GPU path: its time, and the FP32 outputs' error against it."""
    import numpy as np
    p64 = make_problem(mad, mesh, inp, mad.F64, args, stream)
    o64 = p64.outputs()
    mode = mad.ENERGY | mad.GRAD | mad.HESS | mad.SPD
    step_ms, wall = time_steps(torch, lambda: p64.eval(x, mode, out=o64, stream=stream), max(5, args.steps // 5),
                               2, stream)
    ms64 = max(wall * 1e3, sum(step_ms)) / len(step_ms)
    torch.cuda.synchronize()
    e32, g32, h32 = (t.double() for t in out32)
    e64, g64, h64 = o64
    dg = float((g32 - g64).abs().max() / g64.abs().max())
    dh = float((h32 - h64).abs().max() / h64.abs().max())
    de = float(abs(e32[0] - e64[0]) / abs(e64[0]))
    del p64, o64
    return {"ms_per_step_fp64": ms64, "speedup_fp32_over_fp64": ms64 / ms32,
            "grad_max_abs_err_over_max": dg, "hess_max_abs_err_over_max": dh, "energy_rel_err": de}


def per_mesh_baseline(torch, mad, inp, prec, stream, ms_batched, args):
    """The batch as one problem per mesh, evaluated one after another on the same stream."""
    co = inp.comp_offsets
    probs, xs, outs = [], [], []
    for c in range(len(co) - 1):
        lo, hi = int(co[c]), int(co[c + 1])
        import numpy as np
        sel = np.all((inp.tris >= lo) & (inp.tris < hi), axis=1)
        m = mad.Mesh(inp.tris[sel] - lo, hi - lo)
        p = mad.Problem(m, 3, prec)
        for k, prm in SHELL_TERMS:
            p.add_term(k, prm, inp.rest[lo:hi])
        p.finalize(stream)
        probs.append((m, p))
        xs.append(torch.from_numpy(inp.x[lo:hi].ravel().copy()).cuda())
        outs.append(p.outputs())
    mode = mad.ENERGY | mad.GRAD | mad.HESS | mad.SPD

    def step():
        for (m, p), xx, o in zip(probs, xs, outs):
            p.eval(xx, mode, out=o, stream=stream)
    step_ms, wall = time_steps(torch, step, max(3, args.steps // 10), 1, stream)
    ms = max(wall * 1e3, sum(step_ms)) / len(step_ms)
    return {"ms_per_step": ms, "speedup_of_one_launch": ms / ms_batched, "meshes": len(probs)}


if __name__ == "__main__":
    main()
