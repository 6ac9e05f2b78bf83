"""Throughput of the edge-FEM CSEM secondary-field solve on one MI355X.

Default workload (cfg3, the marine layered model at full size): 100^3 x 6 =
6,000,000 jittered tetrahedra, 6,910,300 unknowns, 112,409,452 nonzeros; a
survey of 32 x-dipole positions (x = -3100 + 200 i, z = 50 m) at 0.25, 0.5
and 1.25 Hz (96 sources) and 101 receivers. One step = one pass of the whole
path for one batch of 16 consecutive dipole positions at one frequency: device
re-assembly of K and M_sigma, the 16 right-hand sides, the solve of the
16-column block by COCG preconditioned with multicolour SSOR (`--precond
jacobi` for Jacobi) in complex64 inside complex128 iterative refinement to a
true relative residual of 1e-12, and the total field at the receivers. Timed
step k takes batch k mod 6, so 6 steps cover the survey.
Inputs are resident on the GPU when the timed region starts; host mesh
preprocessing is setup and is reported separately. Beside it: plain FP64
Jacobi GMRES(30) on a stated subset (the centre dipole at each frequency),
and the cfg2 forms.

`value` counts only if every solve converged to its residual and the
sources with stored oracle fields (tests/golden/cfg3_*.npz) match them within
1e-6; otherwise it is null and the line says why. The timed steps themselves
timestamp every sparse-matrix dispatch (HIP events on the solve's stream) for
`roofline` (graphs are off in that mode: the kernels here take milliseconds).

Other workloads (`--workload`):
  cfg2 -- the layered model at 40^3 x 6 = 384,000 tetrahedra, one x-dipole at
          1 Hz: plain GMRES vs mixed COCG, each timed, then a second pass of
          the same steps with per-dispatch timestamps for the roofline.
  cfg4 -- 48 independent models of 1e4..2e6 tetrahedra, one source each, in
          one uneven batch vs plain GMRES one model at a time.
  cfg5 -- the learned initial guess: a network trained on 2000 solves of
          config-1-sized random reservoir models, zero vs learned guess on 200
          held-out seeds (plain GMRES and mixed COCG one seed at a time, and
          the 200 seeds as one uneven batch).
  net  -- the network alone: training steps and forward passes on a batch of
          16, BF16 MFMA throughput against its peak.
  copy -- a 1 GiB device copy (calibration of the rocprofv3 byte counters).
  sync -- the cost of a kernel boundary inside a captured graph against a
          grid barrier inside one persistent cooperative kernel.

    python bench.py [--steps K] [--warmup W] [--gpus 1] [--workload cfg3] [--batch 16]

Prints one JSON line; `cpu_baseline` times the CPU oracle on a bounded
sample of the same workload.
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

HBM_PEAK_GBS = 8000.0
# HBM bytes per launch of the cfg2 sparse kernels from two rocprofv3 --pmc
# passes (FETCH_SIZE, WRITE_SIZE; KiB per dispatch) of the cfg2 bench, scaled
# by the same counters on a 1 GiB device copy (FETCH_SIZE reads 0.5 of the
# bytes copied, WRITE_SIZE 1.0); profiles/spmm_cfg2_traffic.md holds the
# figures and commands. A kernel changed since then reads null.
MEASURED_TRAFFIC = {
    "k_spmm_spb<4, 4> complex64 pipelined sliced ELLPACK with beta partials (K, M_sigma)":
        (49081.9 * 2.0 + 4008.5) * 1024,
    "k_spmm_sp<1, 4> complex64 pipelined sliced ELLPACK (K, M_sigma)": (48342.8 * 2.0 + 3219.3) * 1024,
    "k_spmm_s<1, 4> complex64 sliced ELLPACK (K, M_sigma)": (47676.3 * 2.0 + 3219.2) * 1024,
    "k_spmm_s<1, 8> complex64 sliced ELLPACK (K, M_sigma)": (49890.8 * 2.0 + 3367.3) * 1024,
    # the 6.9M-unknown survey's 8- and 16-column products
    "k_spmm_g<float, 8, 1, 20, 1> complex64 CSR, row entries over the lanes (K, M_sigma) @cfg3":
        (1296681.7 * 2.0 + 435268.0) * 1024,
    "k_spmm_g<float, 8, 2, 20, 1> complex64 CSR, row entries over the lanes (K, M_sigma) @cfg3":
        (1779690.6 * 2.0 + 871820.1) * 1024,
    # its 16-column SSOR blocks in Eisenstat's form: the U sweep, per colour launch
    "k_ssor_eis_u<16, 1> complex64 Eisenstat U sweep with the direction update, one colour per launch "
    "(K, M_sigma) @cfg3": (531263.3 * 2.0 + 244225.6) * 1024,
}
RTOL = 1e-9
# the high-frequency models of the uneven batch (f up to 2 Hz, receivers 4 km
# out where the field has decayed by ~1e-8) need 1e-12: at 1e-10 their far
# receivers still move by up to 1.4e-5, at 3e-11 by up to 2e-6
RTOL_CFG4 = 1e-12
# the survey's end dipoles (x = -3100, 3100 m) have receivers 7.1 km away:
# their per-receiver error against the stored oracle fields was 2.8e-4, 2.5e-5,
# 3.2e-6 and 3.3e-7 at true residuals 1e-9, 1e-10, 1e-11 and 1e-12
RTOL_CFG3 = 1e-12
GOLDEN_CFG2 = os.path.join(ROOT, "tests", "golden", "cfg2_receivers.npz")


def spmv_bytes_fp64(n: int, nnz: int) -> int:
    """Algorithmic bytes of one complex128 CSR SpMV of the GMRES (int32
    indices): value 16 + column 4 per nonzero; x 16 + y 16 + row pointer 4 per
    row."""
    return 20 * nnz + 36 * n


def spmm_bytes_fp32(n: int, nnz: int, cols: int, shape: int = 0) -> int:
    """Algorithmic bytes of one complex64 SpMM of the COCG over real K and
    M_sigma: K, M 4 + 4 and column 4 per nonzero; row pointer 4 per row;
    x read 8, y written 8 per row and column. The single-column product of
    the fused step (shape kind 4) also reads r and D^-1, 8 + 8 per row; the
    per-mesh one (kind 5) r and the two double diagonals, 8 + 16 per row."""
    extra = {4: 16, 5: 24}.get(shape // 10000, 0)
    return 12 * nnz + n * (4 + 16 * cols + extra)


def eis_upass_bytes(S, cols: int) -> int:
    """Algorithmic bytes of one launch of the Eisenstat U pass (one colour of
    the multicolour SSOR; averaged over the colours): per entry coupling a
    row to a later colour its column, K and M_sigma (4 + 4 + 4); per row its
    position, its U range (4 + 4) and the two double diagonals (16); r and p
    read, p and t written, 8 per row and column; and each row of t that the
    colour's rows gather from later colours once, 8 per column."""
    rp, col, _, _ = S.csr()
    color = S.ssor_colors()
    n = len(rp) - 1
    cr = np.repeat(color, np.diff(rp))
    cc = color[col]
    up = cc > cr
    nu = int(up.sum())
    gathered = 0
    for c in range(int(color.max()) + 1):
        gathered += int(np.unique(col[up & (cr == c)]).size)
    total = 12 * nu + n * (4 + 4 + 16) + 4 * n * cols * 8 + gathered * cols * 8
    return total // (int(color.max()) + 1)


def rx_error(E, ref):
    num = np.sqrt(np.sum(np.abs(E - ref) ** 2, axis=-1))
    den = np.sqrt(np.sum(np.abs(ref) ** 2, axis=-1))
    return float(np.max(num / den))


def cpu_baseline_cfg2(model, budget_iters: int):
    """One complete solve of the workload by the CPU oracle (assembly, right-hand
    side, Jacobi GMRES(30) to the same tolerance, receivers), timed on the
    host; `cores` is CPU time over wall time, the threads it actually kept
    busy."""
    from oracle import fem, solve as osolve
    t_cpu0 = time.process_time()
    t0 = time.perf_counter()
    s = fem.assemble(model.xyz, model.tets, model.sigma)
    src = model.sources[0]
    A = fem.system_matrix(s, src.freq)
    b = fem.rhs(model.xyz, model.tets, model.sigma, model.sigma_bg, s.topo, src.pos, src.dir,
                src.freq, src.moment)
    t_setup = time.perf_counter() - t0
    t1 = time.perf_counter()
    x, it, res = osolve.gmres(A, b, rtol=RTOL, restart=30, max_iter=budget_iters)
    t_solve = time.perf_counter() - t1
    t2 = time.perf_counter()
    fem.receivers_total(model.xyz, model.tets, s.topo, x, model.receivers, src.pos, src.dir,
                        src.freq, model.sigma_bg)
    t_rx = time.perf_counter() - t2
    wall = time.perf_counter() - t0
    cores = (time.process_time() - t_cpu0) / wall
    done = res <= RTOL
    per_solve = t_setup + t_rx + (t_solve if done else t_solve / max(it, 1) * budget_iters)
    return {
        "value": 1.0 / per_solve, "unit": "solves/s", "cores": round(cores, 2), "kind": "oracle",
        "sample": (f"one cfg2 solve by the oracle: assembly+RHS {t_setup:.1f} s, Jacobi GMRES(30) "
                   f"{it} iterations to {res:.1e} ({t_solve / max(it, 1) * 1e3:.1f} ms each"
                   f"{'' if done else ', extrapolated to ' + str(budget_iters)}), receivers "
                   f"{t_rx:.1f} s; {wall:.1f} s wall on {len(os.sched_getaffinity(0))} available "
                   f"host cores"),
    }


def kernel_name(form, shape):
    """Name of the sparse kernel a solve used (its spmv_shape stat)."""
    if form == "plain":
        if shape == 1:
            return "k_gm_solve complex128 (A D^-1), all cycles in one launch"
        return f"k_spmv<{shape}, false> complex128 CSR (A D^-1)"
    kind, a, b = shape // 10000, (shape // 100) % 100, shape % 100
    if kind == 7:
        return (f"k_ssor_eis_u<{a}, {b}> complex64 Eisenstat U sweep with the direction update, one colour per "
                f"launch (K, M_sigma)")
    if kind == 5:
        return f"k_spmm_spbs<{b}> complex64 pipelined sliced ELLPACK with beta partials, per mesh (K, M_sigma)"
    if kind == 4:
        return f"k_spmm_spb<{b}, 4> complex64 pipelined sliced ELLPACK with beta partials (K, M_sigma)"
    if kind == 3:
        return f"k_spmm_sp<{a}, {b}> complex64 pipelined sliced ELLPACK (K, M_sigma)"
    if kind == 2:
        return f"k_spmm_s<{a}, {b}> complex64 sliced ELLPACK (K, M_sigma)"
    if kind == 6:
        return f"k_spmm_g<float, {a}, {b}, 20, 1> complex64 CSR, row entries over the lanes (K, M_sigma)"
    if kind == 1:
        return f"k_spmm_n<float, {a}, {b}, 1> complex64 CSR (K, M_sigma)"
    return f"k_spmm_c<float, {a}, {b}, 1> complex64 CSR (K, M_sigma)"


def timed(fn, steps, warmup):
    import torch
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    out = []
    t0 = time.perf_counter()
    for _ in range(steps):
        out.append(fn())
    torch.cuda.synchronize()
    return time.perf_counter() - t0, out


def cfg2_forms(args, petgem, synth, torch, steps, warmup, profile=True):
    """cfg2 (one source): the plain and the mixed form, each over `steps`
    timed steps of the whole path; with `profile` a second pass has every
    sparse-matrix dispatch timestamp its own start and end (no graphs).
    A form counts (`ok`) only if every solve returned OK at the residual and
    its receivers match the stored oracle fields within 1e-6."""
    model = synth.config2()
    t0 = time.perf_counter()
    S = petgem.System.from_model(model)
    setup_s = time.perf_counter() - t0
    sigma_dev = torch.tensor(model.sigma, device="cuda")
    ref = np.load(GOLDEN_CFG2)["E"] if os.path.exists(GOLDEN_CFG2) else None
    forms = {
        "plain": dict(rtol=RTOL),
        "mixed": dict(rtol=RTOL, method=petgem.COCG, precision=petgem.MIXED, inner_rtol=args.inner_rtol,
                      spmm_shape=args.spmm_shape if args.workload == "cfg2" else 0),
    }
    res = {}
    for name, kw in forms.items():
        sol = [None]

        def run(prof):
            opts = petgem.default_opts(profile=prof, **kw)

            def step():
                S.reassemble(sigma_dev, model.sigma_bg)
                sol[0], st, rc = S.solve(model.sources, opts, solution=sol[0], allow_not_converged=True)
                E = sol[0].receivers(model.receivers)
                return st[0], E, rc

            return timed(step, steps, warmup)

        dt, outs = run(0)
        st = [o[0] for o in outs]
        E = outs[-1][1].cpu().numpy()[0]
        converged = all(o[2] == petgem.OK and o[0]["rel_residual"] <= RTOL for o in outs)
        n_launch, avg_ms, dt_prof = 0, float("nan"), None
        if profile:
            dt_prof, pouts = run(1)
            pst = [o[0] for o in pouts]
            n_launch = sum(s["spmv_launches"] for s in pst)
            avg_ms = sum(s["spmv_ms"] for s in pst) / n_launch if n_launch else float("nan")
        nbytes = (spmv_bytes_fp64(S.n_dof, S.nnz) if name == "plain"
                  else spmm_bytes_fp32(S.n_dof, S.nnz, 1, st[-1]["spmv_shape"]))
        err = rx_error(E, ref) if ref is not None else None
        res[name] = {
            "solves_per_s": steps / dt, "ms_per_step": dt / steps * 1e3,
            "iters": st[-1]["iters"], "ir_steps": st[-1]["ir_steps"],
            "rel_residual": st[-1]["rel_residual"], "converged": converged,
            "rx_err_vs_oracle": err, "ok": converged and err is not None and err <= 1e-6,
            # (the profiled pass runs kernel by kernel, and its product is the one timed)
            "kernel": kernel_name(name, (pst if profile else st)[-1]["spmv_shape"]),
            "bytes_per_launch": nbytes, "avg_launch_us": avg_ms * 1e3, "launches": n_launch,
            "profiled_pass_solves_per_s": steps / dt_prof if dt_prof else None,
        }
    res["speedup_mixed_vs_plain"] = res["mixed"]["solves_per_s"] / res["plain"]["solves_per_s"]
    res["setup_s"] = round(setup_s, 3)
    return res, S, model


def bench_cfg2(args, petgem, synth, torch):
    res, S, model = cfg2_forms(args, petgem, synth, torch, args.steps, args.warmup, not args.no_profile)
    ok = [k for k in ("plain", "mixed") if res[k]["ok"]]
    best = max(ok, key=lambda k: res[k]["solves_per_s"]) if ok else "mixed"
    r = res[best]
    achieved = r["bytes_per_launch"] / (r["avg_launch_us"] * 1e-6) / 1e9 if r["launches"] else None
    line = {
        "metric": "receiver-field solves/s at 1e-6 rel err: plain FP64 vs batched/mixed/learned",
        "value": r["solves_per_s"] if ok else None, "unit": "solves/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": r["ms_per_step"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None,
        "dtype": "f64" if best == "plain" else "c64 inner / f64 refinement",
        "data": "synthetic",
        "config": {"workload": "cfg2 marine layered: 384000 jittered tets, 433720 DOF, 6950152 nnz, "
                               "x-dipole 1 Hz, 101 receivers, true relative residual 1e-9",
                   "form": best, "n_dof": S.n_dof, "nnz": S.nnz, "setup_s": res["setup_s"],
                   "tuning": S.tuning(), "parallelism": "1 GPU"},
        "forms": res,
        "speedup_vs_plain": r["solves_per_s"] / res["plain"]["solves_per_s"],
        "roofline": {"kernel": r["kernel"], "bound": "hbm", "achieved": achieved,
                     "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS if achieved else None,
                     "traffic": MEASURED_TRAFFIC.get(r["kernel"]),
                     "bytes_per_launch": r["bytes_per_launch"], "avg_launch_us": r["avg_launch_us"],
                     "launches": r["launches"],
                     "note": "operator (155 MB fp64 / 88 MB fp32) fits the 256 MB Infinity Cache"},
    }
    if not ok:
        line["invalid"] = "no form converged and matched the stored oracle fields within 1e-6"
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline_cfg2(model, 2 * res["plain"]["iters"])
    return line


CFG3_BATCH = 16         # sources per step: a block of consecutive dipole positions at one frequency
CFG3_GOLDEN = {(1.25, 16): "cfg3_f1.25_i16.npz", (1.25, 0): "cfg3_f1.25_i0.npz",
               (0.5, 16): "cfg3_f0.5_i16.npz", (0.25, 16): "cfg3_f0.25_i16.npz"}


def cpu_baseline_cfg3(model, plain_iters: float):
    """The CPU oracle timed on a bounded sample of the cfg3 workload: a slab of
    1/16 of its elements (the first 375,000, x in [-5000, -4375] m, all
    depths) through the oracle's assembly, right-hand side, receiver location
    and 30 iterations of its Jacobi GMRES(30); each part is scaled by 16 (the
    element / nonzero ratio) and the iterations by the iteration count of a
    full cfg3 solve (the plain GMRES(30) subset of this run), assembly
    amortised over the 96 sources that share it. `cores` is CPU time over wall
    time of the sample."""
    from oracle import fem, solve as osolve
    T = len(model.tets) // 16
    tets = model.tets[:T]
    used = np.unique(tets)
    remap = np.full(len(model.xyz), -1, dtype=np.int64)
    remap[used] = np.arange(len(used))
    xyz, tets = model.xyz[used], remap[tets].astype(np.int32)
    sig = model.sigma[:T]
    src = model.sources[2 * 32 + 16]
    rx = model.receivers[model.receivers[:, 0] < -4400.0]
    t_cpu0, t0 = time.process_time(), time.perf_counter()
    s = fem.assemble(xyz, tets, sig)
    t_asm = time.perf_counter() - t0
    t1 = time.perf_counter()
    A = fem.system_matrix(s, src.freq)
    b = fem.rhs(xyz, tets, sig, model.sigma_bg, s.topo, src.pos, src.dir, src.freq, src.moment)
    t_rhs = time.perf_counter() - t1
    t2 = time.perf_counter()
    _, it, _ = osolve.gmres(A, b, rtol=1e-30, restart=30, max_iter=30)
    t_it = (time.perf_counter() - t2) / max(it, 1)
    t3 = time.perf_counter()
    x = np.zeros(s.topo.n_dof, dtype=np.complex128)
    fem.receivers_total(xyz, tets, s.topo, x, rx, src.pos, src.dir, src.freq, model.sigma_bg)
    t_rx = (time.perf_counter() - t3) / max(len(rx), 1) * len(model.receivers)
    wall = time.perf_counter() - t0
    cores = (time.process_time() - t_cpu0) / wall
    per_solve = 16 * (t_asm / 96 + t_rhs + plain_iters * t_it) + 16 * t_rx
    return {
        "value": 1.0 / per_solve, "unit": "solves/s", "cores": round(cores, 2), "kind": "oracle",
        "sample": (f"cfg3 slab of {T} elements ({s.topo.n_dof} unknowns, {A.nnz} nonzeros): oracle assembly "
                   f"{t_asm:.1f} s, RHS {t_rhs:.1f} s, {it} Jacobi GMRES(30) iterations {t_it * 1e3:.0f} ms each, "
                   f"receiver location {t_rx / 16:.2f} s per 101; scaled by 16 and by {plain_iters:.0f} iterations "
                   f"per solve (this run's plain GPU GMRES(30) subset): {per_solve:.0f} s per solve; {wall:.1f} s "
                   f"wall on {len(os.sched_getaffinity(0))} available host cores"),
    }


def bench_cfg3(args, petgem, synth, torch):
    """cfg3: 6,000,000 jittered tetrahedra (6,910,300 unknowns), 96 sources
    (32 dipole positions x 3 frequencies). One step = one batch of B
    consecutive dipole positions at one frequency (B = 16 by default), the whole
    path: device re-assembly of K and M_sigma, the B right-hand sides, the
    mixed-precision COCG solve of the B-column block, the total field at the
    101 receivers. Timed step k takes batch k mod (96 / B), frequency-major,
    so a run of 96 / B steps covers the survey once."""
    model = synth.config3()
    B = args.batch
    nb = len(model.sources) // B
    t0 = time.perf_counter()
    S = petgem.System.from_model(model)
    setup_s = time.perf_counter() - t0
    print(f"cfg3 setup {setup_s:.1f} s (host {S.setup_seconds:.1f} s), {S.n_dof} DOF, {S.nnz} nnz",
          file=sys.stderr, flush=True)
    sigma_dev = torch.tensor(model.sigma, device="cuda")
    o_mix = petgem.default_opts(profile=0 if args.no_profile else 1, rtol=RTOL_CFG3, method=petgem.COCG,
                                precision=petgem.MIXED, inner_rtol=args.inner_rtol, max_iter=args.max_iter,
                                verbose=int(args.verbose), spmm_shape=args.spmm_shape,
                                precond=petgem.SSOR if args.precond == "ssor" else petgem.JACOBI,
                                omega=args.omega)
    sols = {}
    fields = {}       # source index -> receiver total field of its last solve
    bad = []

    def step(k):
        bi = k % nb
        srcs = model.sources[bi * B:(bi + 1) * B]
        S.reassemble(sigma_dev, model.sigma_bg)
        sol, st, rc = S.solve(srcs, o_mix, solution=sols.get(bi), allow_not_converged=True)
        sols[bi] = sol
        E = sol.receivers(model.receivers)
        if rc != petgem.OK or any(s_["rel_residual"] > RTOL_CFG3 for s_ in st):
            bad.append((bi, rc, max(s_["rel_residual"] for s_ in st)))
        print(f"cfg3 step {k}: batch {bi} ({srcs[0].freq} Hz) iters max {max(s_['iters'] for s_ in st)} "
              f"ir {st[0]['ir_steps']} solve {st[0]['t_solve_ms']:.0f} ms", file=sys.stderr, flush=True)
        return bi, st, E

    for k in range(args.warmup):
        step(k)
    torch.cuda.synchronize()
    outs = []
    t0 = time.perf_counter()
    for k in range(args.steps):
        outs.append(step(k))
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    for bi, st, E in outs:
        E = E.cpu().numpy()
        for c in range(B):
            fields[bi * B + c] = E[c]
    n_launch = sum(o[1][0]["spmv_launches"] for o in outs)
    avg_ms = sum(o[1][0]["spmv_ms"] for o in outs) / n_launch if n_launch else float("nan")
    shape = outs[-1][1][0]["spmv_shape"]
    # the profiled kernel: the SpMM, or in Eisenstat's form (no SpMM) its U sweep
    nbytes = eis_upass_bytes(S, B) if shape // 10000 == 7 else spmm_bytes_fp32(S.n_dof, S.nnz, B, shape)
    achieved = nbytes / (avg_ms * 1e-3) / 1e9 if n_launch else None
    kname = kernel_name("mixed", shape)
    # accuracy: every solve converged to RTOL_CFG3 (gate above) and the sources with
    # stored oracle fields match them
    oracle_err = {}
    for (f, i), name in CFG3_GOLDEN.items():
        path = os.path.join(ROOT, "tests", "golden", name)
        k = synth.CFG3_FREQS.index(f) * 32 + i
        if os.path.exists(path) and k in fields:
            oracle_err[f"{f} Hz, x={model.sources[k].pos[0]:.0f}"] = rx_error(fields[k], np.load(path)["E"])
    ok = not bad and all(e <= 1e-6 for e in oracle_err.values())
    # plain FP64 GMRES(30) on a stated subset: the centre dipole at each frequency
    picks = (16,) if args.plain_subset <= 3 else (0, 16, 31)
    sub = [f * 32 + k for f in range(3) for k in picks]
    # (at 1e-12 the 0.25 Hz source needs more than 20,000 GMRES(30) iterations)
    o_plain = petgem.default_opts(rtol=RTOL_CFG3, max_iter=4 * args.max_iter, verbose=int(args.verbose))
    S.solve([model.sources[sub[0]]], o_plain, allow_not_converged=True)   # the plain path's own autotuning
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    psol, pst, prc = S.solve([model.sources[k] for k in sub], o_plain, allow_not_converged=True)
    Ep = psol.receivers(model.receivers)
    torch.cuda.synchronize()
    t_plain = time.perf_counter() - t1
    Ep = Ep.cpu().numpy()
    agree = max((rx_error(fields[k], Ep[i]) for i, k in enumerate(sub) if k in fields), default=None)
    plain_rate = len(sub) / t_plain
    plain_ok = prc == petgem.OK and all(s_["rel_residual"] <= RTOL_CFG3 for s_ in pst)
    value = B * args.steps / dt
    line = {
        "metric": "receiver-field solves/s at 1e-6 rel err: plain FP64 vs batched/mixed/learned",
        "value": value if ok else None, "unit": "solves/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": dt / args.steps * 1e3, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "c64 inner / f64 refinement", "data": "synthetic",
        "config": {"workload": (f"cfg3 marine layered: 6000000 jittered tets, {S.n_dof} DOF, {S.nnz} nnz, 32 x-dipoles "
                                f"x (0.25, 0.5, 1.25) Hz = 96 sources, 101 receivers; one step = {B} dipoles at one "
                                f"frequency as one {B}-column mixed COCG block "
                                f"({'multicolour SSOR' if args.precond == 'ssor' else 'Jacobi'}), true relative "
                                f"residual {RTOL_CFG3:g}"),
                   "form": "batched mixed", "n_dof": S.n_dof, "nnz": S.nnz, "setup_s": round(setup_s, 3),
                   "batch": B, "spmv_shape": shape, "precond": args.precond,
                   "omega": args.omega if args.precond == "ssor" else None, "parallelism": "1 GPU"},
        "accuracy": {"all_converged": not bad, "failures": bad[:5],
                     "rx_err_vs_oracle": oracle_err, "rx_agreement_vs_plain_gpu": agree},
        "plain_subset": {"sources": len(sub), "solves_per_s": plain_rate, "converged": plain_ok,
                         "iters": [s_["iters"] for s_ in pst]},
        "speedup_vs_plain": value / plain_rate,
        "roofline": {"kernel": kname, "bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS if achieved else None,
                     "traffic": MEASURED_TRAFFIC.get(kname + " @cfg3"),
                     "bytes_per_launch": nbytes, "avg_launch_us": avg_ms * 1e3, "launches": n_launch},
    }
    if not ok:
        line["invalid"] = "a solve did not converge or missed 1e-6 against the stored oracle fields"
    if not args.no_cfg2_form:
        del S, sols, psol
        torch.cuda.empty_cache()
        line["forms"] = {"cfg2": cfg2_forms(args, petgem, synth, torch, 5, 1, profile=False)[0]}
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline_cfg3(model, float(np.mean([s_["iters"] for s_ in pst])))
    return line


def bench_cfg4(args, petgem, synth, torch):
    models = synth.config4()
    t0 = time.perf_counter()
    systems = [petgem.System.from_model(m) for m in models]
    setup_s = time.perf_counter() - t0
    srcs = [m.sources[0] for m in models]
    o = petgem.default_opts(rtol=RTOL_CFG4, method=petgem.COCG, precision=petgem.MIXED,
                            inner_rtol=args.inner_rtol, verbose=int(args.verbose))

    def step():
        s_, st, _ = petgem.solve_many(systems, srcs, o)
        Es = [s_[k].receivers(models[k].receivers) for k in range(len(models))]
        return st, Es

    dt, outs = timed(step, args.steps, args.warmup)
    st, Es = outs[-1]
    o_plain = petgem.default_opts(rtol=RTOL_CFG4)
    for Sy, m in zip(systems, models):   # untimed pass: the plain path's own autotuning
        Sy.solve(m.sources, o_plain)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    agree = 0.0
    plain_iters = []
    for k, (Sy, m) in enumerate(zip(systems, models)):
        ps, pst, _ = Sy.solve(m.sources, o_plain)
        E = ps.receivers(m.receivers)
        plain_iters.append(pst[0]["iters"])
        agree = max(agree, rx_error(Es[k].cpu().numpy()[0], E.cpu().numpy()[0]))
    torch.cuda.synchronize()
    t_plain = time.perf_counter() - t1
    value = len(models) * args.steps / dt
    return {
        "metric": "receiver-field solves/s at 1e-6 rel err: plain FP64 vs batched/mixed/learned",
        "value": value, "unit": "solves/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": dt / args.steps * 1e3, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "c64 inner / f64 refinement", "data": "synthetic",
        "config": {"workload": "cfg4: 48 models, 1e4..2e6 tets (log-uniform), one source each, "
                               "one uneven batch, true relative residual 1e-12",
                   "n_tets": [len(m.tets) for m in models],
                   "setup_s": round(setup_s, 3), "iters_max": max(s["iters"] for s in st),
                   "rel_residual_max": max(s["rel_residual"] for s in st), "parallelism": "1 GPU"},
        "plain_sequential": {"solves_per_s": len(models) / t_plain, "iters": plain_iters,
                             "rx_agreement_batched_vs_plain": agree},
        "speedup_vs_plain": value / (len(models) / t_plain),
    }


def bench_cfg5(args, petgem, synth, torch):
    """Learned initial guess: train on solves of config-1-sized random
    reservoir models generated by the library itself, then compare the zero
    and the learned guess on held-out seeds at a true residual of 1e-8."""
    from paper_1808_00186_amd import learned
    mesh = synth.kuhn_mesh(8, -1000.0, 1000.0, 1)
    S = petgem.System.from_model(synth.config5_sample(10000, mesh))
    o_plain = petgem.default_opts(rtol=1e-8)
    o_mix = petgem.default_opts(rtol=1e-8, method=petgem.COCG, precision=petgem.MIXED,
                                inner_rtol=args.inner_rtol)
    g = learned.pilot_scale(S, range(10000, 10016), mesh, o_plain)
    train_seeds = list(synth.CFG5_TRAIN_SEEDS)[: args.n_train]
    data = learned.generate(S, train_seeds, mesh, g, o_plain, progress=250)
    net = petgem.Net(batch_max=16, seed=0)
    t0 = time.perf_counter()
    losses = learned.train(net, data, epochs=args.epochs, batch=16, lr=2e-3, progress=5)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0
    test = list(synth.CFG5_TEST_SEEDS)[: args.n_test]
    forms = {}
    r_plain_E = None
    for name, o in (("plain_fp64_gmres", o_plain), ("mixed_cocg", o_mix)):
        r = learned.evaluate(S, net, test, mesh, g, o)
        if name == "plain_fp64_gmres":
            r_plain_E = r.E_zero
        forms[name] = {
            "zero_guess": {"solves_per_s": len(test) / r.t_zero, "iters_mean": float(np.mean(r.iters_zero))},
            "learned_guess": {"solves_per_s": len(test) / r.t_learned,
                              "iters_mean": float(np.mean(r.iters_learned)),
                              "fallbacks": int(np.sum(r.fallback)),
                              "x0_rel_residual_median": float(np.median(r.x0_residual))},
            "max_rx_diff_learned_vs_zero": r.max_rx_diff,
        }
    # the same held-out seeds as one uneven batch (mixed COCG), zero and learned guesses
    rb = learned.evaluate_batched(net, test, mesh, g, o_mix)
    seq_E = r_plain_E
    forms["batched_mixed_cocg"] = {
        "zero_guess": {"solves_per_s": len(test) / rb.t_zero, "iters_mean": float(np.mean(rb.iters_zero)),
                       "iters_max": int(np.max(rb.iters_zero)), "pass_ms": [round(t * 1e3, 2) for t in rb.t_zero_runs]},
        "learned_guess": {"solves_per_s": len(test) / rb.t_learned,
                          "iters_mean": float(np.mean(rb.iters_learned)),
                          "iters_max": int(np.max(rb.iters_learned)),
                          "fallbacks": int(np.sum(rb.fallback)),
                          "x0_rel_residual_median": float(np.median(rb.x0_residual)),
                          "pass_ms": [round(t * 1e3, 2) for t in rb.t_learned_runs]},
        "max_rx_diff_learned_vs_zero": rb.max_rx_diff,
        "max_rx_diff_vs_sequential_plain": max(rx_error(a, b) for a, b in zip(rb.E_zero, seq_E)),
    }
    plain = forms["plain_fp64_gmres"]["zero_guess"]["solves_per_s"]
    best_name, best = max(((f"{k}/{kk}", v[kk]["solves_per_s"]) for k, v in forms.items()
                           for kk in ("zero_guess", "learned_guess")), key=lambda t: t[1])
    return {
        "metric": "receiver-field solves/s at 1e-6 rel err: plain FP64 vs batched/mixed/learned",
        "value": best, "unit": "solves/s", "n_gpus": 1, "steps": len(test), "warmup": 0,
        "ms_per_step": 1e3 / best, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16 network / c64-f64 solve", "data": "synthetic",
        "config": {"workload": f"cfg5: config-1 mesh with random reservoirs; network trained on {len(train_seeds)} "
                               f"library solves, tested on {len(test)} held-out seeds at residual 1e-8",
                   "best_form": best_name, "g": g, "train_data_s": round(data.seconds, 2),
                   "train_s": round(t_train, 2), "epochs": args.epochs,
                   "loss_first_last": [losses[0], losses[-1]], "parallelism": "1 GPU"},
        "forms": forms, "speedup_vs_plain": best / plain,
    }


NET_LAYERS = ((16, 16, 32), (16, 32, 16), (32, 64, 8), (64, 64, 8), (96, 32, 16), (48, 16, 32), (16, 16, 32))


def bench_net(args, petgem, torch):
    """The learned guess's network alone: training steps (forward, loss,
    backward data and weights, Adam) on a batch of 16 synthetic 32^3 inputs,
    and forward passes; dense BF16 MFMA throughput against the 2.5 PFLOP/s
    peak. FLOPs: 2 x 27 x Cin x Cout x D^3 per convolution and sample; a
    training step counts the forward pass, the weight gradients of every layer
    and the data gradients of all but the first."""
    B = 16
    g = torch.Generator(device="cuda").manual_seed(0)
    x = (torch.randn((B, petgem.NET_VOX, petgem.NET_IN), device="cuda", generator=g) * 0.5).to(torch.bfloat16)
    t = torch.randn((B, petgem.NET_VOX, petgem.NET_OUT_USED), device="cuda", generator=g) * 0.3
    net = petgem.Net(batch_max=B, seed=1)
    conv = [2 * 27 * ci * co * d ** 3 for ci, co, d in NET_LAYERS]
    f_fwd = B * sum(conv)
    f_train = B * (2 * sum(conv) + sum(conv[1:]))
    for _ in range(args.warmup):
        net.train_step(x, t, 1e-4)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        net.train_step(x, t, 1e-4)
    torch.cuda.synchronize()
    dt_train = (time.perf_counter() - t0) / args.steps
    for _ in range(args.warmup):
        net.forward(x)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        net.forward(x)
    torch.cuda.synchronize()
    dt_fwd = (time.perf_counter() - t0) / args.steps
    peak = 2500.0
    return {"metric": "network training samples/s (BF16 MFMA)", "value": B / dt_train, "unit": "samples/s",
            "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": dt_train * 1e3,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16 (fp32 accumulate)",
            "data": "synthetic", "config": {"workload": "3D U-Net on 32^3 voxels, batch 16", "parallelism": "1 GPU"},
            "roofline": {"bound": "mfma", "unit": "TFLOP/s", "peak": peak,
                         "train_achieved": f_train / dt_train / 1e12, "train_frac": f_train / dt_train / 1e12 / peak,
                         "forward_achieved": f_fwd / dt_fwd / 1e12, "forward_frac": f_fwd / dt_fwd / 1e12 / peak,
                         "forward_ms": dt_fwd * 1e3, "flop_per_train_step": f_train, "flop_per_forward": f_fwd}}


def sync_costs(args, petgem):
    """Time per phase separation: a kernel boundary inside a captured graph
    against a grid barrier inside one cooperative (persistent) kernel."""
    out = {"metric": "phase separation cost", "unit": "us per round"}
    for mode, name in ((0, "graph_kernel_boundary"), (1, "grid_barrier_persistent")):
        us, blocks = petgem.sync_probe(2000, mode)
        out[name] = {"us_per_round": us, "blocks": blocks}
    return out


def copy_calibration(args, torch):
    """A plain device copy of a known size (1 GiB read + 1 GiB written per
    launch): the FETCH_SIZE / WRITE_SIZE counters of this kernel give the
    factor that turns the counters of the solver kernels into HBM bytes. Its
    rate (HIP events around each launch, on the stream the copy runs on) is
    the streaming rate a plain kernel reaches, beside the 8 TB/s peak."""
    n = 1 << 30
    a = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(1)
    b = torch.empty_like(a)
    ev = []
    for _ in range(args.steps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        b.copy_(a)
        e1.record()
        ev.append((e0, e1))
    torch.cuda.synchronize()
    ms = [e0.elapsed_time(e1) for e0, e1 in ev]
    best = min(ms[1:] if len(ms) > 1 else ms)
    return {"metric": "copy calibration", "bytes_read_per_launch": n, "bytes_written_per_launch": n,
            "launches": args.steps, "ms_per_launch": ms,
            "best_rate_GBps": 2 * n / (best * 1e-3) / 1e9}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=6)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="cfg3", choices=["cfg2", "cfg3", "cfg4", "cfg5", "net", "copy", "sync"])
    ap.add_argument("--batch", type=int, default=CFG3_BATCH, choices=[1, 2, 4, 8, 16, 32],
                    help="cfg3: sources per step (consecutive dipole positions at one frequency)")
    ap.add_argument("--no-cfg2-form", action="store_true", help="cfg3: skip the cfg2 forms in the line")
    ap.add_argument("--precond", default="ssor", choices=["jacobi", "ssor"],
                    help="cfg3: preconditioner of the mixed COCG (multicolour SSOR or Jacobi)")
    ap.add_argument("--omega", type=float, default=1.0, help="SSOR relaxation factor")
    ap.add_argument("--n-train", type=int, default=2000)
    ap.add_argument("--n-test", type=int, default=200)
    ap.add_argument("--epochs", type=int, default=30)
    ap.add_argument("--inner-rtol", type=float, default=3e-5)
    ap.add_argument("--plain-subset", type=int, default=3, choices=[3, 9],
                    help="cfg3: sources solved by the plain path for the comparison")
    ap.add_argument("--max-iter", type=int, default=20000)
    ap.add_argument("--spmm-shape", type=int, default=0,
                    help="cfg2 / cfg3: force the mixed form's SpMM shape (its spmv_shape code; 0 = "
                         "autotune), so that counter runs measure a chosen kernel")
    ap.add_argument("--verbose", action="store_true")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-profile", action="store_true",
                    help="replay captured graphs without per-launch events (no roofline)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (--gpus {args.gpus} requested); the multi-GPU "
              f"sharding is a design, not a measured path.", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_1808_00186_amd import petgem, synth
    torch.cuda.set_device(0)
    if args.workload == "copy":
        print(json.dumps(copy_calibration(args, torch)), flush=True)
        return
    if args.workload == "sync":
        print(json.dumps(sync_costs(args, petgem)), flush=True)
        return
    if args.workload == "net":
        print(json.dumps(bench_net(args, petgem, torch)), flush=True)
        return
    fn = {"cfg2": bench_cfg2, "cfg3": bench_cfg3, "cfg4": bench_cfg4, "cfg5": bench_cfg5}[args.workload]
    line = fn(args, petgem, synth, torch)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
