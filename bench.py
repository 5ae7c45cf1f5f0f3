#!/usr/bin/env python
"""Benchmark: one shape-optimisation step of differential walk on spheres.

Default workload (N = 1, --workload c3): 3D shape from diffusion -- a
class-I geodesic icosphere of frequency 100 (200,000 triangles) displaced
along the normal by 1024 angular Gaussian bumps with coefficients
N(0, 0.05^2), inside the box [-2, 2]^3, u = 1 on the object and 0 on the
box, sigma = 4, eps = 4e-3, delta = 4e-2, K = 1 nested walk per
differential terminal -- with 65536 query points on the box faces
|coord| = 1.9 x 1024 walks, FP32 walks, gradients with respect to the 1024
coefficients through DWoSFunction.  One step = move the boundary to the
current coefficients (device V(pi) + BVH refit), forward walks (u), squared
loss against a reference solution, backward (differential walks with the
nested forward walks, reverse-mode scatter, SpMV) and an Adam update.

value = walk steps (closest-point queries executed by every forward,
differential and nested walk) per second over the timed steps.  The
roofline object prices the dominant walk kernel's arithmetic against the
FP32 vector peak: the kernel is bound by the issue of divergent vector
instructions, its node and triangle reads being served by the caches.  Their
bytes stand beside it (more than HBM could deliver), with the project's
random-gather probe at the scene's working-set size and, where counters were
taken on the same sources, the traffic beyond the L2.  After the timed window,
at a pinned state (the initial coefficients, independent of --steps), the
second half of the metric: shape-gradient evaluations per second at a fixed
relative RMSE of 0.1, plain walks, the paper's 16 nested walks per terminal
(Table 1) and the learned control variate (the surrogate), and the surrogate's
speedup.

--workload c2 is the 2D screened-Poisson star (4096 segments, 4096 points x
4096 walks, K = 8); the other workloads are listed under --workload.
"""
import argparse
import json
import math
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "walk-steps/s and shape-gradient evals/s at fixed RMSE; surrogate vs plain WoS"

# Algorithmic FP32 operations per counted unit (2D), from the arithmetic of
# the kernels: a pair-node visit evaluates, for both children, a point-box
# squared distance (2 dims x [2 sub, 2 max, 1 fma] = 12) and a point-slab
# squared distance (2 fma, abs-sub, max, mul = 6) plus the max of the two
# (2 x 19 + 2 = 40); a segment test is ~22 (edge/offset differences,
# projection, clamp, residual, squared norm); a walk step adds ~40 (roulette
# scale 1/I0 series, direction, position update); a source sample adds ~200
# (FP64 Green's function series and the Gaussian source) -- counted for
# non-terminal steps only.
OPS_NODE_2D = 40
OPS_PRIM_2D = 22
OPS_STEP_2D = 40
OPS_SOURCE_2D = 200
PEAK_FP32_VALU = 157.3e12     # MI355X FP32 vector, FLOP/s
PEAK_HBM = 8.0e12             # bytes/s
TRAFFIC_FILES = {
    "c2": os.path.join(ROOT, "profiles", "walk_kernel_c2_star4096_hbm.txt"),
    "c3": os.path.join(ROOT, "profiles", "walk_kernel_c3_icosphere200k_hbm.txt"),
    "c4": os.path.join(ROOT, "profiles", "walk_kernel_c4_batch256_hbm.txt"),
}

# Algorithmic bytes per counted unit of the 3D walk kernel: a pair-node visit
# reads both children's boxes and slabs and the two child references (24
# FP32 words, 96 B); a triangle test reads its three vertices (9 FP32 words,
# 36 B; the 12 B that pad the stored record to three 16-byte words are not
# counted).
BYTES_NODE_3D = 96
BYTES_PRIM_3D = 36
# Algorithmic FP32 operations per counted unit (3D), for the ALU side of the
# same kernel: a pair-node visit is two point-box squared distances (3 dims
# x [2 sub, 2 max, 1 fma] = 15) and two point-slab ones (3 fma, abs-sub,
# max, mul = 6) and their maxima (2 x 21 + 2 = 44); a point-triangle test
# ~70 (Voronoi-region classification, Ericson Sec. 5.1.5); a walk step ~100
# (one Philox4x32-10 call, ~40 integer operations, direction, roulette
# scale, position update).
OPS_NODE_3D = 44
OPS_PRIM_3D = 70
OPS_STEP_3D = 100


# the files the walk kernel is compiled from (its build flags are hashed too)
WALK_KERNEL_SOURCES = ["csrc/walk_kernels.hpp", "csrc/device_math.hpp", "csrc/bvh.hpp"]


def sources_sha256():
    """Hash of the walk kernel's sources and compiler flags; HBM counters
    taken on other sources are stale."""
    import hashlib
    from paper_2405_12964_amd import build as hipbuild
    d = os.path.join(ROOT, "paper_2405_12964_amd")
    h = hashlib.sha256()
    for name in WALK_KERNEL_SOURCES:
        with open(os.path.join(d, name), "rb") as f:
            h.update(name.encode() + b"\0" + f.read())
    h.update(" ".join(hipbuild.HIPCC_FLAGS).encode())
    return h.hexdigest()


def walk_kernel_name(dim, kind, stage, cv=False, group=False):
    """The FP32 walk kernel's build: kind 0 forward or 1 differential walks; stage
    0 for a tree read through the caches, 1 for its first nodes in LDS, 2 for all
    of it; with the control variate's records; with lanes that share a walk."""
    return f"walk_kernel<float,{dim},{kind},{stage},{str(cv).lower()},{str(group).lower()}>"


def stage_of(solver):
    """The stage of the solver's walk kernels (see walk_kernel_name)."""
    if solver.get_tuning()["variant"] != 0:
        return 0
    info = solver.scene_info()
    return 2 if info["staged_prims"] and info["staged_nodes"] == info["nodes"] else 1


def measured_traffic(kernel, nested, workload="c2"):
    """Scaled FETCH_SIZE + WRITE_SIZE bytes per launch of `kernel` from the
    committed counter summary of the workload, or None when it is missing or
    was taken on different kernel sources or another nested-walk count.  The
    kernel is looked up by its name or, as the workload fixes the launch's
    shape, by its first three template arguments (type, dimension, kind)."""
    try:
        with open(TRAFFIC_FILES[workload]) as f:
            text = f.read()
    except OSError:
        return None
    kv = dict(re.findall(r"^# (\w+): (\S+)$", text, re.M))
    if kv.get("sources_sha256") != sources_sha256() or kv.get("nested_walks_per_terminal") != str(nested):
        return None
    rows = re.findall(r"^traffic_bytes_per_launch +(\S+) +(\S+)$", text, re.M)
    build = lambda name: name.split(",")[:3]  # noqa: E731
    found = [v for name, v in rows if name == kernel] or [v for name, v in rows if build(name) == build(kernel)]
    return float(found[0]) if found else None


def kernel_ops(tot, has_source=True):
    nonterm = max(0, tot["steps"] - tot["walks"] - tot["nested_walks"])
    return (tot["nodes"] * OPS_NODE_2D + tot["prims"] * OPS_PRIM_2D + tot["steps"] * OPS_STEP_2D
            + (nonterm * OPS_SOURCE_2D if has_source else 0))


def cpu_baseline(sc, X, seed, threads, npts=1024, W=1024, what=""):
    """The FP64 oracle on a bounded sample of the same workload (forward and
    differential walks of npts points x W walks each)."""
    import numpy as np
    import oracle
    o = oracle.Oracle(sc, threads=threads)
    Xs = X[:npts]
    t0 = time.perf_counter()
    _, _, s1 = o.solve(Xs, W, seed)
    w = np.ones(len(Xs))
    _, _, s2 = o.grad(Xs, w, W, seed + 1)
    dt = time.perf_counter() - t0
    return {"value": (s1 + s2) / dt, "unit": "walk-steps/s", "cores": threads, "kind": "oracle",
            "sample": f"{npts} points x {W} forward walks + {npts} x {W} differential walks "
                      f"(K={sc.K} nested) of the same scene ({what}brute-force closest points), FP64, "
                      f"{dt:.1f} s", "walk_steps": int(s1 + s2)}


def run_c5(args):
    """Shape from diffusion on the displaced icosphere (200,000 object
    triangles + box) from c = 0 toward the target coefficients (seed 3),
    with the learned control variate trained online (the surrogate) and with
    plain walks, the same number of iterations each.

    65536 points on the box faces, W forward and W differential walks per
    iteration (W = 64, or annealed geometrically from --walks to
    --c5-final-walks, Sec. 6's walks-per-pixel schedule), squared loss
    against a reference solution of the target coefficients, Adam (lr 1e-3)
    on the 1024 coefficients; in the surrogate run, after each backward, 16
    Adam steps of the control-variate network (16 Fourier frequencies of
    scale 0.125, lr 1e-3) on that iteration's walk records.  The timed
    window is the surrogate run's last --steps iterations.  Progress is
    measured without the walks' own noise: the loss at 1024 walks per point
    with one fixed seed (common to both runs and every evaluation) and the
    coefficient error.  At the surrogate's final coefficients the gradient is
    re-estimated with independent seeds, plain and with the control variate
    at q = 1, 0.5, 0.25, to compare variance x time."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    P, W0 = args.points or 65536, args.walks or 64
    WT = args.c5_final_walks or W0
    iters = args.warmup + args.steps
    nb = 1024
    sc = scenes.c3_icosphere(nu=100, n_basis=nb, coef=np.zeros(nb))
    X = scenes.points_on_box_faces(P, 1)
    Xt = torch.tensor(X, dtype=torch.float64, device=dev)
    coef_t = np.random.default_rng(3).normal(0.0, 0.05, nb)
    ref = dw.Solver.from_scene(sc, "fp32", V=scenes.vertices_at(sc, coef_t))
    uref, _ = ref.solve(Xt, 1024, 99)
    torch.cuda.synchronize()
    del ref
    coef_t_dev = torch.tensor(coef_t, device=dev)

    def walks_at(i):
        # W_t = W_0 exp(log(W_T / W_0) t / T), rounded to a multiple of 8
        w = W0 * math.exp(math.log(WT / W0) * i / max(1, iters - 1))
        return max(8, int(round(w / 8.0)) * 8)

    def optimise(use_cv, timed):
        model = dw.ShapeModel(sc, "fp32")
        net = None
        if use_cv:
            B, th = scenes.mlp_init(3, args.cv_seed, args.cv_freq, args.cv_features)
            th[-(scenes.MLP_WIDTH + 1):] = 0.0        # N = 0: the first calls are plain
            net = dw.Network(3, B, th)
            model.solver.attach_cv(net, 1.0)
        pi = torch.zeros(nb, dtype=torch.float64, device=dev, requires_grad=True)
        opt = torch.optim.Adam([pi], lr=1e-3)

        def true_loss():
            with torch.no_grad():
                model.apply(pi)
                u, _ = model.solver.solve(Xt, 1024, 4242, var=False)
                return float(0.5 * ((u - uref) ** 2).sum().item()), \
                    float(torch.linalg.norm(pi.detach() - coef_t_dev).item())

        def step(i):
            opt.zero_grad(set_to_none=True)
            W = walks_at(i)
            u = dw.DWoSFunction.apply(pi, Xt, model, W, 1000 + 2 * i, W, 1001 + 2 * i)
            loss = 0.5 * ((u - uref) ** 2).sum()
            loss.backward()
            opt.step()
            if use_cv:
                model.solver.cv_train(args.cv_steps, args.cv_batch, args.cv_lr, 50000 + i)
            return loss

        hist = {"iteration": [0], "loss_1024": [], "coef_error": []}
        l0, e0 = true_loss()
        hist["loss_1024"].append(l0)
        hist["coef_error"].append(e0)
        n_pre = args.warmup if timed else iters
        t_all = time.perf_counter()
        for i in range(n_pre):
            step(i)
            if (i + 1) % 50 == 0 and i + 1 < iters:
                l, e = true_loss()
                hist["iteration"].append(i + 1)
                hist["loss_1024"].append(l)
                hist["coef_error"].append(e)
        torch.cuda.synchronize()
        res = {"model": model, "pi": pi, "net": net, "hist": hist}
        if timed:
            for kind in (0, 1):
                model.solver.walk_timing(kind, reset=True)
            t0 = time.perf_counter()
            for i in range(args.steps):
                loss = step(args.warmup + i)
            torch.cuda.synchronize()
            res["elapsed"] = time.perf_counter() - t0
            res["loss"] = float(loss.item())
            res["timing"] = (model.solver.walk_timing(0), model.solver.walk_timing(1))
        res["seconds"] = time.perf_counter() - t_all
        l, e = true_loss()
        hist["iteration"].append(iters)
        hist["loss_1024"].append(l)
        hist["coef_error"].append(e)
        print(f"c5 {'surrogate' if use_cv else 'plain'}: loss_1024 {hist['loss_1024'][0]:.4g} -> {l:.4g}, "
              f"coefficient error {hist['coef_error'][0]:.4f} -> {e:.4f}", file=sys.stderr, flush=True)
        return res

    cvr = optimise(True, True)
    plain = optimise(False, False)
    (ms0, n0, tot0), (ms1, n1, tot1) = cvr["timing"]
    elapsed = cvr["elapsed"]
    model, pi, net = cvr["model"], cvr["pi"], cvr["net"]
    # the same loss at the target coefficients: its floor, the two solutions'
    # own noise at 1024 walks per point
    with torch.no_grad():
        model.apply(coef_t_dev)
        u_t, _ = model.solver.solve(Xt, 1024, 4242, var=False)
        loss_floor = float(0.5 * ((u_t - uref) ** 2).sum().item())

    # gradient variance at the surrogate's final coefficients: plain vs control variate
    with torch.no_grad():
        model.apply(pi)
        u, _ = model.solver.solve(Xt, W0, 777)
        w = (u - uref).contiguous()

    def grads(q, reps=6):
        if q is None:
            model.solver.attach_cv(None)
        else:
            model.solver.attach_cv(net, q)
            model.solver.grad(Xt, w, W0, 900)          # sets beta for this q
        gs, ts = [], []
        for r in range(reps):
            torch.cuda.synchronize()
            t = time.perf_counter()
            g, _ = model.solver.grad(Xt, w, W0, 901 + r, u_mean=False)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
            gs.append(g.cpu().numpy())
        gs = np.array(gs)
        beta = model.solver.cv_beta() if q is not None else None
        return float(gs.var(axis=0, ddof=1).sum()), float(np.mean(ts)), gs.mean(axis=0), beta

    v_plain, t_plain, g_mean, _ = grads(None)
    cv = {"plain": {"grad_var": v_plain, "ms": 1e3 * t_plain}}
    for q in (1.0, 0.5, 0.25):
        v, t, _, beta = grads(q)
        cv[f"q={q}"] = {"grad_var": v, "ms": 1e3 * t, "beta": beta, "var_ratio": v / v_plain,
                        "efficiency": (v_plain * t_plain) / (v * t)}
    steps_total = tot0["steps"] + tot1["steps"]
    pi_np = pi.detach().cpu().numpy()
    hs, hp = cvr["hist"], plain["hist"]
    return {
        "metric": METRIC, "value": steps_total / elapsed, "unit": "walk-steps/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "3D shape from diffusion: displaced icosphere (200,000 triangles) in a "
                               f"box, sigma=4, {P} points x {W0}" + (f"->{WT}" if WT != W0 else "") +
                               f" walks per iteration, {iters} Adam iterations (lr 1e-3) from c = 0 on 1024 "
                               "coefficients, learned control variate trained online", "points": P,
                   "walks_per_point": W0, "final_walks_per_point": WT, "iterations": iters,
                   "triangles": int(sc.prims.shape[0]), "params": nb},
        "grad_evals_per_s": args.steps / elapsed,
        "walk_steps": {"forward": tot0["steps"], "differential": tot1["steps"],
                       "forward_ms": ms0, "differential_ms": ms1},
        "loss": cvr["loss"],
        "surrogate_vs_plain": {
            "loss_1024": {"start": hs["loss_1024"][0], "surrogate": hs["loss_1024"][-1],
                          "plain": hp["loss_1024"][-1], "at_target": loss_floor},
            "coef_error": {"start": hs["coef_error"][0], "surrogate": hs["coef_error"][-1],
                           "plain": hp["coef_error"][-1]},
            "history": {"iteration": hs["iteration"], "surrogate_loss_1024": hs["loss_1024"],
                        "plain_loss_1024": hp["loss_1024"], "surrogate_coef_error": hs["coef_error"],
                        "plain_coef_error": hp["coef_error"]},
            "seconds": {"surrogate": cvr["seconds"], "plain": plain["seconds"]},
            "loss_1024_note": "0.5 sum (u - uref)^2 with u from 1024 walks per point, one fixed seed",
        },
        "grad_norm": float(np.linalg.norm(g_mean)),
        # cosine between the descent direction and the way to the target
        "grad_alignment": float(-g_mean @ (coef_t - pi_np) /
                                (np.linalg.norm(g_mean) * np.linalg.norm(coef_t - pi_np))),
        "cv_training": {"freq_scale": args.cv_freq, "features": args.cv_features, "init_seed": args.cv_seed,
                        "adam_steps_per_iteration": args.cv_steps, "batch": args.cv_batch, "lr": args.cv_lr},
        "control_variate": cv,
    }


def run_c4(args):
    """Many instances of uneven size in one persistent launch: 256 displaced
    icospheres in boxes (980 - 100,820 triangles, log-uniform), 512 - 16384
    points each (log-uniform), screening sigma_i ~ U(0, 20), W walks per
    point.  One step = the batched forward solve of every instance and the
    batched reverse mode (each instance's 256 radial-basis coefficients, K =
    1), captured once in a hipGraph on the context stream and replayed with a
    new device seed per step, after the autotuner has set the walk kernels'
    scheduling knobs for the batch.  Beside it: the same two calls issued
    eagerly (their walk-kernel times give the roofline), and the forward work
    as one context and one launch per instance."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    W = args.walks or 64
    insts = scenes.c4_batch()
    if args.calib_copy_mb:
        a = torch.empty(args.calib_copy_mb * (1 << 20) // 4, dtype=torch.float32, device=dev).fill_(1.0)
        b = a.clone()
        torch.cuda.synchronize()
        del a, b
    stream = torch.cuda.Stream()
    s = dw.Solver(3, "fp32", stream=stream)
    sc0 = insts[0][0]
    s.set_problem(dw.make_problem(0.0, sc0.eps, sc0.delta, 1, sc0.kmax, 1, 0.0, None, sc0.bc, 3))
    for i, (sc, _) in enumerate(insts):
        s.batch_add_instance(sc.V, sc.prims, sc.label, sc.sigma, sc.eps, sc.delta)
        s.batch_set_parameters(i, sc.N, sc.rowptr, sc.pid, sc.vel)
    X = torch.tensor(np.concatenate([x for _, x in insts]), dtype=torch.float64, device=dev)
    P = [len(x) for _, x in insts]
    wts = torch.cat([torch.full((len(x),), 1.0 / len(x), dtype=torch.float64, device=dev) for _, x in insts])
    with torch.cuda.stream(stream):
        s.batch_solve(X, P, W, 1, var=False)
        tuning, tune_ms = (s.get_tuning(), None) if args.no_autotune else s.autotune(X, W, seed=5, P=P, cache=False, grad=True)
        s.batch_grad(X, P, wts, W, 2, u_mean=False)
    torch.cuda.synchronize()
    print(f"c4: {len(insts)} instances, tuning {tuning} ({tune_ms} ms)", file=sys.stderr, flush=True)

    def eager(i):
        s.batch_solve(X, P, W, 10 + i, var=False)
        s.batch_grad(X, P, wts, W, 20 + i, u_mean=False)

    with torch.cuda.stream(stream):
        for i in range(args.warmup):
            eager(i)
    torch.cuda.synchronize()
    for kind in (0, 1):
        s.walk_timing(kind, reset=True)
    t0 = time.perf_counter()
    with torch.cuda.stream(stream):
        for i in range(args.steps):
            eager(i)
    torch.cuda.synchronize()
    elapsed_eager = time.perf_counter() - t0
    ms0, n0, tot0 = s.walk_timing(0)
    ms1, n1, tot1 = s.walk_timing(1)

    # the step captured once and replayed with a new device seed each time
    seed_buf = torch.zeros(1, dtype=torch.int64, device=dev)
    s.set_seed_buffer(seed_buf)
    with torch.cuda.stream(stream):
        eager(0)   # an identical call before the capture: tables and workspaces in place
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        eager(0)
    with torch.cuda.stream(stream):
        for i in range(args.warmup):
            seed_buf.fill_(1000 + i)
            graph.replay()
    torch.cuda.synchronize()
    for kind in (0, 1):
        s.walk_timing(kind, reset=True)
    t1 = time.perf_counter()
    with torch.cuda.stream(stream):
        for i in range(args.steps):
            seed_buf.fill_(2000 + i)
            graph.replay()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t1
    _, _, gt0 = s.walk_timing(0)
    _, _, gt1 = s.walk_timing(1)
    s.set_seed_buffer(None)
    for t in (tot0, tot1, gt0, gt1):
        assert t["stack_overflow"] == 0 and t["invalid"] == 0, t
    steps_total = gt0["steps"] + gt1["steps"]

    # the forward work as one context and one launch per instance
    solvers = []
    for (sc, x) in insts:
        si = dw.Solver(3, "fp32")
        si.set_boundary(sc.V, sc.prims, sc.label, sc.gvert)
        si.set_problem(dw.make_problem(sc.sigma, sc.eps, sc.delta, 1, sc.kmax, 1, 0.0, None, sc.bc, 3))
        solvers.append((si, torch.tensor(x, dtype=torch.float64, device=dev)))
    for si, xi in solvers:
        si.solve(xi, W, 1, var=False)
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    for i in range(args.steps):
        for si, xi in solvers:
            si.solve(xi, W, 10 + i, var=False)
    torch.cuda.synchronize()
    elapsed_seq = time.perf_counter() - t2
    fwd_eager_s = ms0 / 1e3
    del solvers

    kind, ms, n, tot = (1, ms1, n1, tot1) if ms1 >= ms0 else (0, ms0, n0, tot0)
    # (batches stage nothing: every instance has its own tree)
    kname = walk_kernel_name(3, kind, 1 if tuning["variant"] == 0 else 0)
    info = s.scene_info()
    roof = roofline_3d(kname, ms, n, tot, measured_traffic(kname, 1, "c4"), info)
    out = {
        "metric": METRIC, "value": steps_total / elapsed, "unit": "walk-steps/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": f"256 instances (displaced icospheres in boxes, 980-100,820 triangles, 512-16384 "
                               f"points, sigma ~ U(0,20), 256 radial-basis coefficients each): batched forward "
                               f"solve + batched reverse mode (K = 1), W = {W}, one hipGraph replay per step",
                   "instances": len(insts), "triangles": int(sum(sc.prims.shape[0] for sc, _ in insts)),
                   "points": int(sum(P)), "walks_per_point": W, "params": int(sum(sc.N for sc, _ in insts))},
        "tuning": tuning, "autotune_ms": tune_ms,
        "walk_steps": {"forward": gt0["steps"], "differential": gt1["steps"], "nested_walks": gt1["nested_walks"]},
        "eager": {"ms_per_step": 1e3 * elapsed_eager / args.steps,
                  "forward_kernel_ms": ms0 / max(1, n0), "differential_kernel_ms": ms1 / max(1, n1),
                  "walk_steps_per_s": (tot0["steps"] + tot1["steps"]) / elapsed_eager},
        "per_instance_launches": {"forward_ms_per_step": 1e3 * elapsed_seq / args.steps,
                                  "batched_forward_kernel_ms": 1e3 * fwd_eager_s / max(1, n0),
                                  "speedup_of_one_launch": (elapsed_seq / args.steps) / (fwd_eager_s / max(1, n0))},
        "roofline": roof,
    }
    if not args.no_cpu_baseline:
        import oracle
        threads = min(16, len(os.sched_getaffinity(0)))
        t3 = time.perf_counter()
        st = 0
        for sc, x in insts[:4]:
            o = oracle.Oracle(sc, threads=threads)
            _, _, s1 = o.solve(x[:64], 16, 7)
            st += s1
        dt = time.perf_counter() - t3
        out["cpu_baseline"] = {"value": st / dt, "unit": "walk-steps/s", "cores": threads, "kind": "oracle",
                               "sample": f"instances 0-3 x 64 points x 16 forward walks, brute-force FP64, "
                                         f"{dt:.1f} s", "walk_steps": int(st)}
    return out


def run_c5ls(args):
    """Shape from diffusion with the paper's optimiser for mesh vertices:
    the 200,000-triangle icosphere starts undisplaced, the target is the
    displaced sphere of coefficient seed 3; every object vertex coordinate is
    a parameter (300,006 in all).  One iteration: forward walks at 65536
    points on the box faces, squared loss, reverse-mode differential walks,
    one vector-Adam step on (I + lambda L) x with the max second moment
    (lambda 20, lr 1e-3, two CG solves), BVH refit; walks per point annealed
    from 8 to 64 over 200 iterations (eq. update_rule).  The timed window is
    iterations [warmup, warmup + steps) of that schedule; one periodic remesh
    of the object is timed after it."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw
    from paper_2405_12964_amd.shapeopt import VertexShapeOptimizer

    dev = torch.device("cuda:0")
    P = args.points or 65536
    T_iters = 200
    start = scenes.c3_icosphere(coef_std=0.0)
    target = scenes.c3_icosphere(coef_seed=3)
    X = torch.tensor(scenes.points_on_box_faces(P, 1), dtype=torch.float64, device=dev)
    ref = dw.Solver.from_scene(target, "fp32")
    uref, _ = ref.solve(X, 256, 99)
    torch.cuda.synchronize()
    del ref
    print("reference solution done", file=sys.stderr, flush=True)
    nb = 8
    mv = np.concatenate([np.zeros(nb, bool), np.ones(start.nv - nb, bool)])
    opt = VertexShapeOptimizer(start, mv, lam=20.0, lr=1e-3, W0=8, WT=64, T=T_iters)
    losses = []
    for i in range(args.warmup):
        L, W, its = opt.step(X, uref, 1000 + i)
        losses.append(L)
        print(f"warmup iteration {i}: loss {L:.4f} W {W} cg {its}", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    for kind in (0, 1):
        opt.solver.walk_timing(kind, reset=True)
    cg = []
    t0 = time.perf_counter()
    for i in range(args.steps):
        L, W, its = opt.step(X, uref, 1000 + args.warmup + i)
        losses.append(L)
        cg.append(its)
        print(f"iteration {args.warmup + i}: loss {L:.4f} W {W} cg {its}", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms0, n0, tot0 = opt.solver.walk_timing(0)
    ms1, n1, tot1 = opt.solver.walk_timing(1)
    steps_total = tot0["steps"] + tot1["steps"]
    # the periodic remesh (every 100 iterations in the paper), timed once
    # after the window: host isotropic remeshing of the object toward its
    # initial mean edge length, then the boundary, Jacobian and optimiser
    # rebuilt on the new mesh
    nf0 = len(opt.P)
    t0 = time.perf_counter()
    opt.remesh()
    torch.cuda.synchronize()
    remesh_s = time.perf_counter() - t0
    return {
        "metric": METRIC, "value": steps_total / elapsed, "unit": "walk-steps/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "shape from diffusion, 200,000-triangle icosphere, all 300,006 object vertex "
                               f"coordinates as parameters, {P} points on the box faces, walks per point "
                               "annealed 8 -> 64 over 200 iterations, vector Adam on (I + 20 L) x with the "
                               "max second moment", "points": P, "params": int(3 * (start.nv - nb))},
        "walk_ms_per_iteration": (ms0 + ms1) / args.steps,
        "cg_iterations": cg,
        "loss": {"first": losses[0], "last": losses[-1]},
        "remesh": {"seconds": remesh_s, "iterations": opt.remesh_iters, "target_edge": opt.remesh_len,
                   "triangles_before": nf0, "triangles_after": int(len(opt.P))},
    }


def run_thermal(args):
    """Walk on stars: one optimisation step of the 2D thermal-design stand-in
    (four heating wires of 125 segments, g = 1, 64 shape coefficients; a fixed
    zero-flux slice of 65,536 segments between them; a cold box, Laplace).
    16384 points on the slice surface, where the loss lives, with their walks
    starting on the wall; W forward and W differential walks (K nested walks
    on stars at each wire terminal, --nested, 8 as in the paper's thermal
    design); squared loss against the solution of a second coefficient draw;
    Adam on the coefficients."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    P, W = args.points or 16384, args.walks or 256
    sc = scenes.thermal_scene(K=8 if args.nested is None else args.nested)
    X, seg = scenes.points_on_segments(sc.NV, sc.nsegs, P, 1)
    Xt = torch.tensor(X, dtype=torch.float64, device=dev)
    ref = dw.Solver.from_scene(scenes.thermal_scene(coef_seed=3), "fp32")
    ref.set_start_segments(seg)
    uref, _ = ref.solve(Xt, W, 99)
    torch.cuda.synchronize()
    print("reference solution done", file=sys.stderr, flush=True)
    del ref
    model = dw.ShapeModel(sc, "fp32")
    model.solver.set_start_segments(seg)
    pi = torch.tensor(sc.pi0, dtype=torch.float64, device=dev, requires_grad=True)
    opt = torch.optim.Adam([pi], lr=1e-3)

    def step(i):
        opt.zero_grad(set_to_none=True)
        u = dw.DWoSFunction.apply(pi, Xt, model, W, 1000 + 2 * i, W, 1001 + 2 * i)
        loss = 0.5 * ((u - uref) ** 2).sum()
        loss.backward()
        opt.step()
        return loss

    for i in range(args.warmup):
        step(i)
        torch.cuda.synchronize()
        print(f"warmup step {i} done", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    for kind in (0, 1):
        model.solver.walk_timing(kind, reset=True)
    t0 = time.perf_counter()
    for i in range(args.steps):
        loss = step(args.warmup + i)
        print(f"step {i} queued", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms0, n0, tot0 = model.solver.walk_timing(0)
    ms1, n1, tot1 = model.solver.walk_timing(1)
    assert tot0["stack_overflow"] == 0 and tot1["stack_overflow"] == 0
    assert tot0["invalid"] == 0 and tot1["invalid"] == 0
    kind, ms, n, tot = (1, ms1, n1, tot1) if ms1 >= ms0 else (0, ms0, n0, tot0)
    avg_s = ms / max(1, n) / 1e3
    ops = kernel_ops(tot, has_source=False) / max(1, n)
    out = {
        "metric": METRIC, "value": (tot0["steps"] + tot1["steps"]) / elapsed, "unit": "walk-steps/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "walk on stars, 2D thermal design: 4 heating wires (500 segments, g = 1, "
                               "64 shape coefficients), zero-flux slice of 65,536 segments, cold box, "
                               f"Laplace; {P} points on the slice x {W} walks, forward + differential "
                               f"(K={sc.K} nested) via autograd",
                   "points": P, "walks_per_point": W, "reflecting_segments": int(len(sc.nsegs)),
                   "dirichlet_segments": int(len(sc.prims)), "params": int(sc.N)},
        "grad_evals_per_s": args.steps / elapsed,
        "walk_steps": {"forward": tot0["steps"], "differential": tot1["steps"],
                       "forward_ms": ms0, "differential_ms": ms1,
                       "truncated": tot0["truncated"] + tot1["truncated"]},
        "loss": float(loss.item()),
        "roofline": {"bound": "alu", "achieved": ops / avg_s / 1e12, "peak": PEAK_FP32_VALU / 1e12,
                     "unit": "TFLOP/s", "frac": ops / avg_s / PEAK_FP32_VALU, "traffic": None,
                     "kernel": f"wost_kernel<float,{kind}>", "avg_launch_ms": ms / max(1, n),
                     "launches": n, "ops_per_launch": ops,
                     "steps_per_launch": tot["steps"] / max(1, n),
                     "nodes_per_step": tot["nodes"] / max(1, tot["steps"]),
                     "prims_per_step": tot["prims"] / max(1, tot["steps"])},
    }
    if not args.no_cpu_baseline:
        import oracle
        threads = min(16, len(os.sched_getaffinity(0)))
        o = oracle.Oracle(sc, threads=threads)
        npts, Wc = 64, 64
        t0 = time.perf_counter()
        _, _, s1 = o.solve(X[:npts], Wc, 7, start_seg=seg[:npts])
        _, _, s2 = o.grad(X[:npts], np.ones(npts), Wc, 8, start_seg=seg[:npts])
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": (s1 + s2) / dt, "unit": "walk-steps/s", "cores": threads,
                               "kind": "oracle",
                               "sample": f"{npts} points x {Wc} forward + {Wc} differential walks on stars "
                                         f"(K = {sc.K} nested) "
                                         f"of the same scene, brute-force FP64, {dt:.1f} s"}
    return out


def run_thermal3d(args):
    """Walk on stars in 3D: one optimisation step of the 3D thermal-design
    stand-in (four heating elements, displaced icospheres of 720 triangles,
    g = 1, 64 shape coefficients; a fixed zero-flux superellipsoid slice of
    64,980 triangles between them; a cold box, Laplace).  Points on the slice
    surface, where the loss lives, with their walks starting on the wall; W
    forward and W differential walks (K nested walks on stars at each element
    terminal, 8 as in the paper's thermal design); squared loss against the
    solution of a second coefficient draw; Adam on the coefficients."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    P, W = args.points or 16384, args.walks or 64
    K = 8 if args.nested is None else args.nested
    sc = scenes.thermal3d_scene(K=K)
    X, tri = scenes.points_on_triangles(sc.NV, sc.nsegs, P, 1)
    Xt = torch.tensor(X, dtype=torch.float64, device=dev)
    ref = dw.Solver.from_scene(scenes.thermal3d_scene(coef_seed=3), "fp32")
    ref.set_start_segments(tri)
    uref, _ = ref.solve(Xt, W, 99)
    torch.cuda.synchronize()
    print("reference solution done", file=sys.stderr, flush=True)
    del ref
    model = dw.ShapeModel(sc, "fp32")
    model.solver.set_start_segments(tri)
    pi = torch.tensor(sc.pi0, dtype=torch.float64, device=dev, requires_grad=True)
    opt = torch.optim.Adam([pi], lr=1e-3)

    def step(i):
        opt.zero_grad(set_to_none=True)
        u = dw.DWoSFunction.apply(pi, Xt, model, W, 1000 + 2 * i, W, 1001 + 2 * i)
        loss = 0.5 * ((u - uref) ** 2).sum()
        loss.backward()
        opt.step()
        return loss

    for i in range(args.warmup):
        step(i)
        torch.cuda.synchronize()
        print(f"warmup step {i} done", file=sys.stderr, flush=True)
    for kind in (0, 1):
        model.solver.walk_timing(kind, reset=True)
    t0 = time.perf_counter()
    for i in range(args.steps):
        loss = step(args.warmup + i)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms0, n0, tot0 = model.solver.walk_timing(0)
    ms1, n1, tot1 = model.solver.walk_timing(1)
    for t in (tot0, tot1):
        assert t["stack_overflow"] == 0 and t["invalid"] == 0, t
    kind, ms, n, tot = (1, ms1, n1, tot1) if ms1 >= ms0 else (0, ms0, n0, tot0)
    avg_s = ms / max(1, n) / 1e3
    bytes_launch = (tot["nodes"] * BYTES_NODE_3D + tot["prims"] * BYTES_PRIM_3D) / max(1, n)
    out = {
        "metric": METRIC, "value": (tot0["steps"] + tot1["steps"]) / elapsed, "unit": "walk-steps/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "walk on stars, 3D thermal design: 4 heating elements (2,880 triangles, g = 1, "
                               "64 shape coefficients), zero-flux superellipsoid slice of 64,980 triangles, cold "
                               f"box, Laplace; {P} points on the slice x {W} walks, forward + differential "
                               f"(K={sc.K} nested) via autograd",
                   "points": P, "walks_per_point": W, "reflecting_triangles": int(len(sc.nsegs)),
                   "dirichlet_triangles": int(len(sc.prims)), "params": int(sc.N)},
        "grad_evals_per_s": args.steps / elapsed,
        "walk_steps": {"forward": tot0["steps"], "differential": tot1["steps"],
                       "forward_ms": ms0, "differential_ms": ms1,
                       "truncated": tot0["truncated"] + tot1["truncated"]},
        "loss": float(loss.item()),
        "roofline": {"bound": "hbm", "achieved": bytes_launch / avg_s / 1e9, "peak": PEAK_HBM / 1e9,
                     "unit": "GB/s", "frac": bytes_launch / avg_s / PEAK_HBM, "traffic": None,
                     "kernel": f"wost3_kernel<float,{kind}>", "avg_launch_ms": ms / max(1, n),
                     "launches": n, "algorithmic_bytes_per_launch": bytes_launch,
                     "steps_per_launch": tot["steps"] / max(1, n),
                     "nodes_per_step": tot["nodes"] / max(1, tot["steps"]),
                     "prims_per_step": tot["prims"] / max(1, tot["steps"])},
    }
    if not args.no_cpu_baseline:
        import oracle
        threads = min(16, len(os.sched_getaffinity(0)))
        o = oracle.Oracle(sc, threads=threads)
        npts, Wc = 16, 8
        t0 = time.perf_counter()
        _, _, s1 = o.solve(X[:npts], Wc, 7, start_seg=tri[:npts])
        _, _, s2 = o.grad(X[:npts], np.ones(npts), Wc, 8, start_seg=tri[:npts])
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": (s1 + s2) / dt, "unit": "walk-steps/s", "cores": threads,
                               "kind": "oracle",
                               "sample": f"{npts} points x {Wc} forward + {Wc} differential walks on stars "
                                         f"(K = {sc.K} nested) of the same scene, brute-force FP64, {dt:.1f} s"}
    return out


# Algorithmic FP32 operations per step of a walk on the implicit boundary of
# n monopoles: h and grad h (per monopole: 2 differences, squared norm 3,
# sqrt, a/r, accumulate, a/r^3 with 2 products, 4 for the gradient = 15),
# the Newton steps of the direct safe radius counting each |x - p_n| once
# (per monopole and step: r + d, a/q, add, q^2, a/q^2, add = 6; five steps,
# where the iteration has converged to FP32 resolution for 99.9% of the
# positions of the inflation scene), the nearest pole (1 per monopole), and
# ~40 for the Harnack radius, roulette, direction and position update.
def imp_ops_per_step(n):
    return 15 * n + 5 * 6 * n + n + 40


def run_inflation(args):
    """Curve inflation (Sec. 7.4) on an implicit boundary: 32 harmonic
    monopoles (c = -1), -Lap u = 4, g = 0, 128 x 128 pixel centres on
    [-1, 1]^2, W = 4 differential walks per pixel with K = 4 nested walks,
    eps = 1e-3, delta = 1e-2 (the paper's table row for this example); the
    loss is over the whole image, the height being 0 outside the domain.
    One iteration (ImplicitShapeOptimizer): the pixel regions, the
    squared-loss U-statistic gradient over the pixels inside the domain
    beyond the band (all W walks of a pixel form one batch), W forward walks
    at the band pixels (band eps_band = 2 pixels; a second context and stream,
    overlapping the differential walks) for the band term with
    integrand l(u) - uref^2/2, Adam on the 96 monopole coordinates with the
    scales kept >= 1e-3, and the new monopoles uploaded.  The rate counts
    the steps of both kinds of walks."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    side = int(round(math.sqrt(args.points))) if args.points else 128
    W = args.walks or 4
    g1 = -1.0 + (np.arange(side) + 0.5) * 2.0 / side
    X = np.stack(np.meshgrid(g1, g1), -1).reshape(-1, 2)
    dA = (2.0 / side) ** 2
    eps_band = 2 * 2.0 / side
    Xt = torch.tensor(X, dtype=torch.float64, device=dev)
    target = scenes.inflation_scene(32, seed=1).with_(K=4)
    start = scenes.inflation_scene(32, seed=2).with_(K=4)
    ref = dw.Solver.from_scene(target, "fp32")
    zero = torch.zeros(len(X), dtype=torch.float64, device=dev)
    _, reg = ref.implicit_band_grad(Xt, zero, eps_band, want_mask=True)
    inside = torch.nonzero(reg > 0).squeeze(1)
    uref = torch.zeros(len(X), dtype=torch.float64, device=dev)
    uref[inside] = ref.solve(Xt[inside].contiguous(), 256, 99)[0]
    torch.cuda.synchronize()
    del ref
    print("reference heightfield done", file=sys.stderr, flush=True)
    from paper_2405_12964_amd.shapeopt import ImplicitShapeOptimizer
    opt = ImplicitShapeOptimizer(start, Xt, uref, dA, eps_band, lr=2e-3, W=W, a_min=1e-3)
    s = opt.solver

    def step(i):
        return opt.step(5000 + i)

    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()
    print(f"{args.warmup} warmup iterations done", file=sys.stderr, flush=True)
    sb = opt.band_solver
    sb.walk_timing(0, reset=True)
    s.walk_timing(1, reset=True)
    npx = []
    t0 = time.perf_counter()
    for i in range(args.steps):
        loss, n_in = step(args.warmup + i)
        npx.append(n_in)
        if i % 50 == 49:
            print(f"iteration {i + 1} done", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms0, n0, tot0 = sb.walk_timing(0)
    ms1, n1, tot1 = s.walk_timing(1)
    assert tot0["invalid"] == 0 and tot1["invalid"] == 0
    n = len(start.mono)
    avg_s = ms1 / max(1, n1) / 1e3
    ops = tot1["steps"] * imp_ops_per_step(n) / max(1, n1)
    out = {
        "metric": METRIC, "value": (tot0["steps"] + tot1["steps"]) / elapsed, "unit": "walk-steps/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"curve inflation on an implicit boundary: {n} harmonic monopoles (c = -1), "
                               f"-Lap u = 4, g = 0; {side}x{side} pixels on [-1,1]^2, {W} differential walks "
                               f"per pixel inside the domain (K = 4 nested), squared-loss U-statistic + "
                               f"band term ({W} forward walks per band pixel), Adam on the {3 * n} monopole coordinates",
                   "pixels": side * side, "walks_per_point": W, "monopoles": n, "params": 3 * n,
                   "mean_pixels_inside": float(np.mean(npx))},
        "grad_evals_per_s": args.steps / elapsed,
        "walk_steps": {"differential": tot1["steps"], "differential_ms": ms1, "walks": tot1["walks"],
                       "forward_band": tot0["steps"], "forward_band_ms": ms0,
                       "nested_walks": tot1["nested_walks"], "truncated": tot1["truncated"]},
        "loss": float(loss),
        "roofline": {"bound": "alu", "achieved": ops / avg_s / 1e12, "peak": PEAK_FP32_VALU / 1e12,
                     "unit": "TFLOP/s", "frac": ops / avg_s / PEAK_FP32_VALU, "traffic": None,
                     "kernel": "implicit_kernel<float,1>", "avg_launch_ms": ms1 / max(1, n1),
                     "launches": n1, "ops_per_launch": ops, "ops_per_step": imp_ops_per_step(n),
                     "steps_per_launch": tot1["steps"] / max(1, n1)},
    }
    if not args.no_cpu_baseline:
        import oracle
        threads = min(16, len(os.sched_getaffinity(0)))
        o = oracle.Oracle(start.with_(mono=opt.mono), threads=threads)
        reg = opt.regions().cpu().numpy()
        sel = np.nonzero(reg == 2)[0][:8192]
        Wc = 256
        t0 = time.perf_counter()
        _, _, _, st = o.grad_sqloss(X[sel], uref.cpu().numpy()[sel], Wc, 4, 7)
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": st / dt, "unit": "walk-steps/s", "cores": threads, "kind": "oracle",
                               "sample": f"{len(sel)} pixels inside the domain x {Wc} differential walks "
                                         f"(K = 4 nested, batches of 4) at the final monopoles, squared-loss "
                                         f"U-statistic, brute-force FP64, {dt:.1f} s"}
    return out


def run_adjoint(args):
    """Ablation of Appendix B: the adjoint formulation against the
    differential walks on the same derivative.  Unit disk as a 1024-gon,
    -Lap u = 4, g = 0, eps = 1e-4, delta = 1e-2; J = int 1/2 (u - uref)^2
    with uref = c0 (1 - |x|^2), c0 = 1/2 (zero on the boundary, so neither
    formulation has a boundary term), pi = R, dJ/dR = pi (1 - c0) exactly.
      differential: P points uniform in the domain x W walks (the
        squared-loss U-statistic over each point's W walks) times |Omega|/P;
      adjoint: S boundary samples x W walks (dwos_adjoint_grad).
    Each is repeated with independent seeds; reported per formulation: time
    and walk steps per gradient, RMSE against the exact value, and
    time x RMSE^2 (the time to reach unit variance).  value = walk steps per
    second of the adjoint kernel."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    n, c0 = 1024, 0.5
    sc = scenes.c1_polygon(n, eps=1e-4, delta=1e-2).with_(bc=[scenes._restricted(0.0, dim=2)], src_c0=4.0)
    exact = math.pi * (1 - c0)
    P = S = args.points or 16384
    W = args.walks or 8
    reps = args.steps
    s = dw.Solver.from_scene(sc, "fp32")
    # differential walks over the domain: points at least 2e-3 inside (a walk
    # started within rounding of the boundary has no defined side); the band
    # left out holds ~1e-5 of the integral, whose integrand vanishes on the
    # boundary
    rmax = math.cos(math.pi / n) - 2e-3
    X = scenes.points_in_disk(P, rmax, 5)
    Xt = torch.tensor(X, dtype=torch.float64, device=dev)
    uref_p = torch.tensor(c0 * (1 - (X ** 2).sum(1)), dtype=torch.float64, device=dev)
    area = math.pi * rmax * rmax
    # adjoint: boundary samples
    code, bary, wq = scenes.boundary_samples(sc, S, 6)
    ct = torch.tensor(code, dtype=torch.int32, device=dev)
    bt = torch.tensor(bary, dtype=torch.float64, device=dev)
    wt = torch.tensor(wq, dtype=torch.float64, device=dev)
    uref_q = (c0, None, np.diag([-c0, -c0]))

    def diff(seed):
        _, g, _, st = s.grad_sqloss(Xt, uref_p, W, W, seed, stats=True)
        return float(g[0]) * area / P, st["steps"]

    def adj(seed):
        g, st = s.adjoint_grad(ct, bt, wt, uref_q, W, seed, stats=True)
        return float(g[0]), st["steps"]

    out = {}
    for name, fn in (("differential", diff), ("adjoint", adj)):
        for i in range(args.warmup):
            fn(10 + i)
        torch.cuda.synchronize()
        for kind in (1, 2):
            s.walk_timing(kind, reset=True)
        vals, steps, t = [], 0, 0.0
        for r in range(reps):
            t0 = time.perf_counter()
            v, st = fn(1000 + r)
            torch.cuda.synchronize()
            t += time.perf_counter() - t0
            vals.append(v)
            steps += st
        print(f"{name}: {reps} gradients done", file=sys.stderr, flush=True)
        vals = np.array(vals)
        rmse = float(np.sqrt(np.mean((vals - exact) ** 2)))
        kind = 1 if name == "differential" else 2
        kms, kn, ktot = s.walk_timing(kind)
        out[name] = {"ms_per_grad": 1e3 * t / reps, "walk_steps_per_grad": steps / reps,
                     "rmse": rmse, "rel_rmse": rmse / exact, "mean": float(vals.mean()),
                     "bias": float(vals.mean() - exact), "ms_x_rmse2": 1e3 * t / reps * rmse ** 2,
                     "kernel_ms_per_grad": kms / max(1, kn), "kernel_totals": ktot}
    d, a = out["differential"], out["adjoint"]
    ktot = a["kernel_totals"]
    avg_s = a["kernel_ms_per_grad"] / 1e3
    ops = kernel_ops(ktot)
    res = {
        "metric": METRIC, "value": ktot["steps"] / max(1e-12, ktot["walk_ms"] / 1e3), "unit": "walk-steps/s",
        "n_gpus": 1, "steps": reps, "warmup": args.warmup,
        "ms_per_step": a["ms_per_grad"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"adjoint ablation (Appendix B): unit disk as a {n}-gon, -Lap u = 4, g = 0, "
                               f"uref = {c0} (1 - |x|^2), d/dR; differential walks at {P} interior points "
                               f"x {W} walks vs the adjoint at {S} boundary samples x {W} walks, "
                               f"eps 1e-4, delta 1e-2",
                   "points": P, "samples": S, "walks_per_point": W, "exact": exact},
        "ablation": {"differential": {k: v for k, v in d.items() if k != "kernel_totals"},
                     "adjoint": {k: v for k, v in a.items() if k != "kernel_totals"},
                     "steps_ratio": a["walk_steps_per_grad"] / d["walk_steps_per_grad"],
                     "cost_to_variance_ratio": a["ms_x_rmse2"] / d["ms_x_rmse2"]},
        "roofline": {"bound": "alu", "achieved": ops / max(1e-12, ktot["walk_ms"] / 1e3) / 1e12,
                     "peak": PEAK_FP32_VALU / 1e12, "unit": "TFLOP/s",
                     "frac": ops / max(1e-12, ktot["walk_ms"] / 1e3) / PEAK_FP32_VALU, "traffic": None,
                     "kernel": "adjoint_kernel<float,2>", "avg_launch_ms": a["kernel_ms_per_grad"],
                     "steps_per_launch": ktot["steps"] / max(1, reps)},
    }
    if not args.no_cpu_baseline:
        import oracle
        threads = min(16, len(os.sched_getaffinity(0)))
        o = oracle.Oracle(sc, threads=threads)
        Sc = 1024
        ref = np.concatenate([[c0], np.zeros(2), np.diag([-c0, -c0]).ravel()])
        t0 = time.perf_counter()
        _, _, _, st = o.adjoint_grad(code[:Sc], bary[:Sc], wq[:Sc], ref, W, 7)
        dt = time.perf_counter() - t0
        res["cpu_baseline"] = {"value": float(st.sum()) / dt, "unit": "walk-steps/s", "cores": threads,
                               "kind": "oracle",
                               "sample": f"{Sc} boundary samples x {W} adjoint walks with their nested "
                                         f"forward walks, brute-force FP64, {dt:.1f} s"}
    return res


def probe_gather(ws_bytes):
    """The project's random-gather probe (dwos_probe_bandwidth): GB/s of
    random 64-byte gathers over a buffer of the walk kernel's working-set
    size, of the same gathers over 4 GiB (HBM-resident), and of a streaming
    read of 4 GiB."""
    import ctypes as C
    from paper_2405_12964_amd import capi

    def run(nbytes, line, mode):
        g, ms = C.c_double(), C.c_double()
        capi.check(capi.dwos_probe_bandwidth(int(nbytes), int(line), int(mode), C.byref(g), C.byref(ms)))
        return g.value

    ws = max(1 << 16, int(ws_bytes))
    return {"working_set_bytes": ws,
            "gather64_working_set_GBs": run(ws, 64, 0),
            "gather64_4GiB_GBs": run(4 << 30, 64, 0),
            "stream_4GiB_GBs": run(4 << 30, 64, 1)}


def roofline_3d(kname, ms, n, tot, traffic, info):
    """The roofline object of a 3D walk kernel: n launches of ms in all with the
    counters tot; traffic: bytes beyond the L2 per launch, or None; info: the
    scene's sizes."""
    n = max(1, n)
    avg_s = ms / n / 1e3
    bytes_launch = (tot["nodes"] * BYTES_NODE_3D + tot["prims"] * BYTES_PRIM_3D) / n
    ops_launch = (tot["nodes"] * OPS_NODE_3D + tot["prims"] * OPS_PRIM_3D + tot["steps"] * OPS_STEP_3D) / n
    # the scene's node and primitive arrays: what the traversals gather from
    probe = probe_gather(info["node_bytes"] + info["prim_bytes"])
    return {"bound": "alu", "achieved": ops_launch / avg_s / 1e12, "peak": PEAK_FP32_VALU / 1e12,
            "unit": "TFLOP/s", "frac": ops_launch / avg_s / PEAK_FP32_VALU, "traffic": traffic,
            "hbm_frac": traffic / avg_s / PEAK_HBM if traffic else None,
            "kernel": kname, "avg_launch_ms": ms / n, "launches": n, "ops_per_launch": ops_launch,
            "steps_per_launch": tot["steps"] / n,
            "nodes_per_step": tot["nodes"] / max(1, tot["steps"]),
            "prims_per_step": tot["prims"] / max(1, tot["steps"]),
            "scene": info,
            "cache_reads": {"algorithmic_bytes_per_launch": bytes_launch,
                            "bytes_per_step": bytes_launch / max(1.0, tot["steps"] / n),
                            "GBs": bytes_launch / avg_s / 1e9, "gather_probe": probe}}


def grad_rmse_rate(solver, Xt, w, target=0.1, W_probe=256, reps=12, seed0=60000, W_time_max=4096):
    """Shape-gradient evaluations per second at a fixed relative RMSE.

    The reverse-mode gradient g = sum_p w_p udot(x_p) (dwos_grad, fixed
    weights w) is unbiased, so its RMSE about the exact gradient g* is the
    root of its variance.  `reps` independent gradients at W_probe walks per
    point give the per-parameter variance (ddof 1) and, from their mean, the
    bias-corrected ||g*||^2 = mean(gbar^2) - var/reps.  With variance ~ 1/W,
    the walks per point that reach RMSE = target ||g*||_RMS are
    W* = W_probe (rel_rmse / target)^2.  The time per gradient is measured at
    min(W*, W_time_max) walks per point and scaled linearly in W beyond it
    (a gradient at W walks runs ceil(P W / 2^26) identical launches)."""
    import numpy as np
    import torch
    gs, ts = [], []
    solver.grad(Xt, w, W_probe, seed0 - 1, u_mean=False)
    for r in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        g, _ = solver.grad(Xt, w, W_probe, seed0 + r, u_mean=False)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t0)
        gs.append(g.cpu().numpy())
    G = np.array(gs)
    var = G.var(axis=0, ddof=1)
    mse = float(var.mean())
    gstar2 = float(np.mean(G.mean(axis=0) ** 2) - var.mean() / reps)
    if not gstar2 > 0:
        return {"error": "gradient not resolved above its noise at the probe", "mse_at_probe": mse}
    rel = math.sqrt(mse / gstar2)
    Wstar = max(1, int(math.ceil(W_probe * (rel / target) ** 2)))
    Wt = min(Wstar, W_time_max)
    solver.grad(Xt, w, Wt, seed0 + 1000, u_mean=False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for r in range(2):
        solver.grad(Xt, w, Wt, seed0 + 1001 + r, u_mean=False)
    torch.cuda.synchronize()
    t = (time.perf_counter() - t0) / 2 * (Wstar / Wt)
    return {"target_rel_rmse": target, "walks_per_point": Wstar, "grad_evals_per_s": 1.0 / t,
            "ms_per_grad": 1e3 * t, "timed_walks_per_point": Wt, "extrapolated": Wstar > Wt,
            "rel_rmse_at_probe": rel, "probe_walks_per_point": W_probe, "probe_replicates": reps,
            "ms_per_grad_at_probe": 1e3 * float(np.median(ts)),
            "grad_rms": math.sqrt(gstar2),
            # relative standard error of the ||g*|| estimate from the pooled replicates
            "grad_rms_rel_se": 0.5 * rel / math.sqrt(reps)}


def run_c3(args):
    """The default workload: 3D shape from diffusion on the 200,000-triangle
    displaced icosphere, 65536 box-face points x 1024 walks, gradients with
    respect to the 1024 coefficients through DWoSFunction (see the module
    docstring)."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    P, W = args.points or 65536, args.walks or 1024
    K = args.nested if args.nested is not None else 1
    nb = 1024
    sc = scenes.c3_icosphere(nu=100, n_basis=nb, coef_seed=0, K=K)
    X = scenes.points_on_box_faces(P, 1)
    Xt = torch.tensor(X, dtype=torch.float64, device=dev)
    print(f"scene: {sc.prims.shape[0]} triangles, {P} points", file=sys.stderr, flush=True)

    if args.calib_copy_mb:
        a = torch.empty(args.calib_copy_mb * (1 << 20) // 4, dtype=torch.float32, device=dev).fill_(1.0)
        b = a.clone()
        torch.cuda.synchronize()
        del a, b

    # reference solution at the target coefficients (seed 3; setup, untimed)
    coef_t = np.random.default_rng(3).normal(0.0, 0.05, nb)
    ref = dw.Solver.from_scene(sc, "fp32", V=scenes.vertices_at(sc, coef_t))
    uref, _ = ref.solve(Xt, W, 99, var=False)
    torch.cuda.synchronize()
    del ref
    print("reference solution done", file=sys.stderr, flush=True)

    model = dw.ShapeModel(sc, "fp32")
    pi = torch.tensor(sc.pi0, dtype=torch.float64, device=dev, requires_grad=True)
    opt = torch.optim.Adam([pi], lr=1e-3)

    def step(i):
        opt.zero_grad(set_to_none=True)
        u = dw.DWoSFunction.apply(pi, Xt, model, W, 1000 + 2 * i, W, 1001 + 2 * i)
        loss = 0.5 * ((u - uref) ** 2).sum()
        loss.backward()
        opt.step()
        return loss

    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()
    print(f"{args.warmup} warmup steps done", file=sys.stderr, flush=True)
    for kind in (0, 1):
        model.solver.walk_timing(kind, reset=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        loss = step(args.warmup + i)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    print(f"{args.steps} timed steps done", file=sys.stderr, flush=True)
    ms0, n0, tot0 = model.solver.walk_timing(0)
    ms1, n1, tot1 = model.solver.walk_timing(1)
    for t in (tot0, tot1):
        assert t["stack_overflow"] == 0 and t["invalid"] == 0 and t["truncated"] == 0, t
    steps_total = tot0["steps"] + tot1["steps"]
    kind, ms, n, tot = (1, ms1, n1, tot1) if ms1 >= ms0 else (0, ms0, n0, tot0)
    kname = walk_kernel_name(3, kind, stage_of(model.solver))
    roof = roofline_3d(kname, ms, n, tot, measured_traffic(kname, K, "c3"), model.solver.scene_info())
    out = {
        "metric": METRIC, "value": steps_total / elapsed, "unit": "walk-steps/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "3D shape from diffusion: displaced icosphere (200,000 triangles, 1024 "
                               "radial-basis coefficients N(0,0.05^2)) in the box [-2,2]^3, u=1 on the object, "
                               f"0 on the box, sigma=4, eps=4e-3, delta=4e-2; {P} box-face points x {W} walks, "
                               f"grads wrt the 1024 coefficients via autograd (forward walks + differential "
                               f"walks, K={K} nested)",
                   "points": P, "walks_per_point": W, "triangles": int(sc.prims.shape[0]), "params": nb,
                   "nested_walks_per_terminal": K},
        "grad_evals_per_s": args.steps / elapsed,
        "walk_steps": {"forward": tot0["steps"], "differential": tot1["steps"],
                       "forward_ms": ms0, "differential_ms": ms1,
                       "forward_walks": tot0["walks"], "differential_walks": tot1["walks"],
                       "nested_walks": tot1["nested_walks"]},
        "loss": float(loss.item()),
        "roofline": roof,
    }
    if not args.no_fixed_rmse:
        out["fixed_rmse"] = c3_fixed_rmse(args, sc, Xt, uref)
    if not args.no_cpu_baseline:
        threads = min(16, len(os.sched_getaffinity(0)))
        out["cpu_baseline"] = cpu_baseline(sc, X, 7, threads, npts=args.cpu_points or 64, W=args.cpu_walks or 16,
                                           what="full 200,000-triangle mesh, ")
    return out


def c3_fixed_rmse(args, sc, Xt, uref):
    """The metric's second half at a pinned state: the initial coefficients
    (seed 0) and fixed weights w = u - uref (u from 1024 walks per point,
    seed 777), independent of the timed steps.  Three estimators of the same
    gradient: plain walks with K = 1 nested walk per terminal, the paper's
    Table 1 setting of 16 nested walks, and the learned control variate of
    the nested walks (q = 1, trained online at this state on earlier walks
    only).  Reported per estimator: walks per point for a relative RMSE of
    0.1 and gradient evaluations per second there; and the surrogate's
    speedup at equal RMSE over plain walks."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    s = dw.Solver.from_scene(sc.with_(K=1), "fp32")
    u, _ = s.solve(Xt, 1024, 777, var=False)
    w = (u - uref).contiguous()
    res = {"state": "initial coefficients (seed 0), w = u(1024 walks, seed 777) - uref",
           "estimator": "reverse mode sum_p w_p udot(x_p), fixed w"}
    res["plain"] = grad_rmse_rate(s, Xt, w, W_probe=args.probe_walks, seed0=60000)
    print("fixed-RMSE plain done", file=sys.stderr, flush=True)
    s16 = dw.Solver.from_scene(sc.with_(K=16), "fp32")
    res["nested16"] = grad_rmse_rate(s16, Xt, w, W_probe=args.probe_walks, seed0=70000)
    del s16
    print("fixed-RMSE K=16 done", file=sys.stderr, flush=True)
    # the surrogate: the control-variate network trained online at this state
    B, th = scenes.mlp_init(3, args.cv_seed, args.cv_freq, args.cv_features)
    th[-(scenes.MLP_WIDTH + 1):] = 0.0        # N = 0: the first calls are plain
    net = dw.Network(3, B, th)
    s.attach_cv(net, 1.0)
    t0 = time.perf_counter()
    for i in range(args.cv_iters):
        s.grad(Xt, w, args.cv_walks, 80000 + i, u_mean=False)
        s.cv_train(args.cv_steps, args.cv_batch, args.cv_lr, 90000 + i)
    torch.cuda.synchronize()
    train_s = time.perf_counter() - t0
    cv = grad_rmse_rate(s, Xt, w, W_probe=args.probe_walks, seed0=100000)
    cv["beta"] = s.cv_beta()
    cv["training"] = {"iterations": args.cv_iters, "walks_per_point": args.cv_walks,
                      "adam_steps_per_iteration": args.cv_steps, "batch": args.cv_batch, "lr": args.cv_lr,
                      "frequencies": args.cv_features, "freq_scale": args.cv_freq, "init_seed": args.cv_seed,
                      "seconds": train_s}
    res["control_variate"] = cv
    print("fixed-RMSE control variate done", file=sys.stderr, flush=True)
    p = res["plain"]
    if "ms_per_grad" in p and "ms_per_grad" in cv:
        res["surrogate_speedup_at_equal_rmse"] = p["ms_per_grad"] / cv["ms_per_grad"]
    if "ms_per_grad" in p and "ms_per_grad" in res["nested16"]:
        res["nested16_speedup_at_equal_rmse"] = p["ms_per_grad"] / res["nested16"]["ms_per_grad"]
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None)
    ap.add_argument("--warmup", type=int, default=None)
    ap.add_argument("--workload", choices=["c3", "c2", "c4", "c5", "c5ls", "thermal", "thermal3d", "inflation",
                                           "adjoint"],
                    default="c3",
                    help="c3: 3D shape from diffusion on the 200,000-triangle icosphere (the reported "
                         "configuration); c2: 2D star; c4: batched instances; c5: 3D shape from diffusion "
                         "with the learned control variate; c5ls: 3D shape from diffusion with vertex "
                         "parameters and the preconditioned vector Adam; thermal: walk on stars with a "
                         "reflecting boundary; inflation: curve inflation on an implicit boundary of harmonic "
                         "monopoles; adjoint: the adjoint formulation of Appendix B against the differential "
                         "walks")
    ap.add_argument("--points", type=int, default=0)
    ap.add_argument("--nested", type=int, default=None,
                    help="nested forward walks per differential terminal (K): c3 1, c2 and thermal 8 "
                         "(the paper uses 2-16, 8 for its thermal design)")
    ap.add_argument("--walks", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true", help="skip the oracle timing")
    ap.add_argument("--no-fixed-rmse", action="store_true",
                    help="c3, c2: skip the gradient rate at fixed RMSE (and the control variate's speedup)")
    ap.add_argument("--probe-walks", type=int, default=256,
                    help="c3, c2: walks per point of the replicate gradients that measure the RMSE")
    ap.add_argument("--cpu-points", type=int, default=0, help="c3: points of the oracle's sample (64)")
    ap.add_argument("--cpu-walks", type=int, default=0, help="c3: walks per point of the oracle's sample (16)")
    ap.add_argument("--cv-freq", type=float, default=0.125, help="c3, c5: Fourier frequency scale")
    ap.add_argument("--cv-features", type=int, default=16, help="c3, c5: Fourier frequencies (2F + 3 <= 64)")
    ap.add_argument("--cv-steps", type=int, default=16, help="c3, c5: network Adam steps per iteration")
    ap.add_argument("--cv-batch", type=int, default=8192, help="c3, c5: walks per network Adam step")
    ap.add_argument("--cv-lr", type=float, default=1e-3, help="c3, c5: network learning rate")
    ap.add_argument("--cv-seed", type=int, default=4, help="c3, c5: network initialisation seed")
    ap.add_argument("--cv-iters", type=int, default=100,
                    help="c3: training iterations of the control variate at the pinned state")
    ap.add_argument("--cv-walks", type=int, default=64,
                    help="c3: walks per point of each training iteration's differential call")
    ap.add_argument("--no-autotune", action="store_true", help="c4: keep the default scheduling knobs")
    ap.add_argument("--c5-final-walks", type=int, default=0,
                    help="c5: anneal the walks per point geometrically from --walks to this count")
    ap.add_argument("--calib-copy-mb", type=int, default=0,
                    help="run a plain device copy of this size first (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "the benchmark runs on one GPU; the walks shard across GPUs "
                                   "by (point, walk) ranges but no multi-GPU path is built",
                          "n_gpus": args.gpus}))
        sys.exit(2)

    if args.workload == "c4":
        args.steps = 5 if args.steps is None else args.steps
        args.warmup = 2 if args.warmup is None else args.warmup
        print(json.dumps(run_c4(args)), flush=True)
        return
    if args.workload == "c5ls":
        args.steps = 10 if args.steps is None else args.steps
        args.warmup = 20 if args.warmup is None else args.warmup
        print(json.dumps(run_c5ls(args)), flush=True)
        return
    if args.workload == "thermal":
        args.steps = 5 if args.steps is None else args.steps
        args.warmup = 2 if args.warmup is None else args.warmup
        print(json.dumps(run_thermal(args)), flush=True)
        return
    if args.workload == "thermal3d":
        args.steps = 3 if args.steps is None else args.steps
        args.warmup = 1 if args.warmup is None else args.warmup
        print(json.dumps(run_thermal3d(args)), flush=True)
        return
    if args.workload == "inflation":
        args.steps = 150 if args.steps is None else args.steps
        args.warmup = 10 if args.warmup is None else args.warmup
        print(json.dumps(run_inflation(args)), flush=True)
        return
    if args.workload == "adjoint":
        args.steps = 16 if args.steps is None else args.steps
        args.warmup = 1 if args.warmup is None else args.warmup
        print(json.dumps(run_adjoint(args)), flush=True)
        return
    if args.workload == "c5":
        args.steps = 50 if args.steps is None else args.steps
        args.warmup = 150 if args.warmup is None else args.warmup
        print(json.dumps(run_c5(args)), flush=True)
        return
    if args.workload == "c2":
        args.steps = 5 if args.steps is None else args.steps
        args.warmup = 2 if args.warmup is None else args.warmup
        args.nested = 8 if args.nested is None else args.nested
        print(json.dumps(run_c2(args)), flush=True)
        return
    args.steps = 5 if args.steps is None else args.steps
    args.warmup = 2 if args.warmup is None else args.warmup
    print(json.dumps(run_c3(args)), flush=True)


def run_c2(args):
    """2D screened-Poisson star: 4096 segments, 4096 points x 4096 walks,
    K nested walks (--nested, 8 by default), gradients with respect to the 64
    Fourier coefficients through DWoSFunction."""
    import numpy as np
    import torch
    import scenes
    import paper_2405_12964_amd as dw

    dev = torch.device("cuda:0")
    P, W = args.points or 4096, args.walks or 4096
    sc = scenes.c2_star(n=4096, coef_seed=0, K=args.nested)
    X = scenes.star_points(P, 1)
    Xt = torch.tensor(X, dtype=torch.float64, device=dev)

    if args.calib_copy_mb:
        a = torch.empty(args.calib_copy_mb * (1 << 20) // 4, dtype=torch.float32, device=dev).fill_(1.0)
        b = a.clone()
        torch.cuda.synchronize()
        del a, b

    # reference solution at the target coefficients (setup, untimed)
    coef_t = scenes.star_coefficients(3)
    ref = dw.Solver.from_scene(sc, "fp32", V=scenes.vertices_at(sc, coef_t))
    uref, _ = ref.solve(Xt, W, 99)
    torch.cuda.synchronize()
    del ref

    model = dw.ShapeModel(sc, "fp32")
    pi = torch.tensor(sc.pi0, dtype=torch.float64, device=dev, requires_grad=True)
    opt = torch.optim.Adam([pi], lr=1e-3)

    def step(i):
        opt.zero_grad(set_to_none=True)
        u = dw.DWoSFunction.apply(pi, Xt, model, W, 1000 + 2 * i, W, 1001 + 2 * i)
        loss = 0.5 * ((u - uref) ** 2).sum()
        loss.backward()
        opt.step()
        return loss

    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()
    for kind in (0, 1):
        model.solver.walk_timing(kind, reset=True)

    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        loss = step(args.warmup + i)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    elapsed = t1 - t0

    ms0, n0, tot0 = model.solver.walk_timing(0)
    ms1, n1, tot1 = model.solver.walk_timing(1)
    steps_total = tot0["steps"] + tot1["steps"]
    value = steps_total / elapsed
    # dominant kernel: the differential walk kernel (or whichever took longer)
    kind, ms, n, tot = (1, ms1, n1, tot1) if ms1 >= ms0 else (0, ms0, n0, tot0)
    avg_s = ms / max(1, n) / 1e3
    ops = kernel_ops(tot) / max(1, n)
    achieved = ops / avg_s
    kname = walk_kernel_name(2, kind, stage_of(model.solver))
    roof = {"bound": "alu", "achieved": achieved / 1e12, "peak": PEAK_FP32_VALU / 1e12,
            "unit": "TFLOP/s", "frac": achieved / PEAK_FP32_VALU, "traffic": measured_traffic(kname, args.nested, "c2"),
            "kernel": kname, "avg_launch_ms": ms / max(1, n),
            "launches": n, "ops_per_launch": ops,
            "steps_per_launch": tot["steps"] / max(1, n),
            "nodes_per_step": tot["nodes"] / max(1, tot["steps"]),
            "prims_per_step": tot["prims"] / max(1, tot["steps"])}
    assert tot0["stack_overflow"] == 0 and tot1["stack_overflow"] == 0
    assert tot0["invalid"] == 0 and tot1["invalid"] == 0

    out = {
        "metric": METRIC, "value": value, "unit": "walk-steps/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "2D screened Poisson star polygon, 4096 segments, sigma=10, "
                               f"Gaussian source, {P} points x {W} walks, grads wrt 64 coeffs "
                               f"via autograd (forward walks + differential walks, K={args.nested} nested)",
                   "points": P, "walks_per_point": W, "segments": 4096, "params": 64,
                   "nested_walks_per_terminal": args.nested},
        "grad_evals_per_s": args.steps / elapsed,
        "walk_steps": {"forward": tot0["steps"], "differential": tot1["steps"],
                       "forward_ms": ms0, "differential_ms": ms1},
        "loss": float(loss.item()),
        "roofline": roof,
    }
    if not args.no_cpu_baseline:
        out["fixed_rmse"] = c2_fixed_rmse(args, sc, Xt, uref)
        threads = min(16, len(os.sched_getaffinity(0)))
        # a sample of ~20 s: 1024 points at K = 1, fewer as the nested walks grow
        npts = max(128, 1024 // max(1, (args.nested + 1) // 2) * 2)
        out["cpu_baseline"] = cpu_baseline(sc, X, 7, threads, npts=min(1024, npts))
    return out




def c2_fixed_rmse(args, sc, Xt, uref):
    """Gradient evaluations per second at a fixed relative RMSE of 0.1 on the
    star, at a pinned state: the initial coefficients (seed 0) and weights
    w = u - uref with u from 4096 walks per point (seed 777)."""
    import paper_2405_12964_amd as dw
    s = dw.Solver.from_scene(sc, "fp32")
    u, _ = s.solve(Xt, 4096, 777, var=False)
    w = (u - uref).contiguous()
    res = grad_rmse_rate(s, Xt, w, W_probe=args.probe_walks, seed0=60000)
    res["state"] = "initial coefficients (seed 0), w = u(4096 walks, seed 777) - uref"
    return res


if __name__ == "__main__":
    main()
