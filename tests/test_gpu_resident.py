"""The resident COCG (one kernel per inner solve) against the library's own
double-precision right-hand side and product, and its iteration counts
against the kernel-per-phase form. Marked `gpu`.

The true residual |b - A x| / |b| of every column is formed from
``System.rhs`` and ``System.spmv``, each pinned to the oracle by its own test,
so its bound is the solve's tolerance itself (1 % for the rounding of the
residual's own evaluation). The two forms run the same recurrence in exact
arithmetic; their roundings moved iteration counts by up to 10 %, so the
bound on them is 25 % and one check interval.
"""
import numpy as np
import pytest

from paper_1808_00186_amd import synth

pytestmark = pytest.mark.gpu

RTOL = 1e-10


@pytest.fixture(scope="module")
def pg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1808_00186_amd import petgem
    petgem.lib()
    return petgem


def _model(n, seed=5, f=1.0, box=3000.0):
    xyz, tets = synth.kuhn_mesh(n, -box, box, seed + n)
    sig = synth.marine_sigma(synth.centroids(xyz, tets), ((-0.4 * box, 0.4 * box), (-0.4 * box, 0.4 * box),
                                                          (-0.6 * box, -0.2 * box)), 0.02)
    return synth.Model(f"resident-{n}", xyz, tets, sig, 3.3, [synth.Dipole((30.0, 0.0, 50.0), f)],
                       np.zeros((1, 3)), n, (-box, box))


def _residuals(S, srcs, x):
    b = S.rhs(srcs)
    r = [b[k] - S.spmv(d.freq, x[k].contiguous()) for k, d in enumerate(srcs)]
    return [float(r[k].norm() / b[k].norm()) for k in range(len(srcs))]


# 2: 26 unknowns, most lanes idle; 5: 665, two workgroups, the second partly
# filled; 8: 6 workgroups; 16: 52, two levels of sums; 23: 158 (nine columns
# of it: the coarser split, in turn on its domains)
@pytest.mark.parametrize("n", [2, 5, 8, 16, 23])
@pytest.mark.parametrize("cols", [1, 2, 9])
def test_resident_columns_reach_the_true_residual(pg, n, cols):
    print(f"[case] resident n={n} cols={cols}", flush=True)
    m = _model(n)
    S = pg.System.from_model(m)
    srcs = [synth.Dipole((-200.0 + 90.0 * k, 10.0, 50.0 + 5 * k), (0.5, 1.3, 2.0)[k % 3]) for k in range(cols)]
    o = pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL)
    sol, st, rc = S.solve(srcs, o)
    assert rc == pg.OK
    res = _residuals(S, srcs, sol.x())
    print(f"  iters {[s['iters'] for s in st]} residual {max(res):.1e}", flush=True)
    assert max(res) <= 1.01 * RTOL
    again, _, _ = S.solve(srcs, o)
    assert np.array_equal(sol.x().cpu().numpy(), again.x().cpu().numpy())
    # a chosen shape runs kernel by kernel
    k = pg.spmm_candidates(cols, cols <= 4)[-1]
    _, stk, _ = S.solve(srcs, pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL, spmm_shape=k))
    for a, b in zip(st, stk):
        assert a["iters"] <= 1.25 * b["iters"] + 8


def test_more_columns_than_resident_domains(pg):
    """70 columns of a mesh that the coarser split gives 12 workgroups: 21 are
    resident together, the others follow on the same workgroups."""
    m = _model(14)
    S = pg.System.from_model(m)
    srcs = [synth.Dipole((-700.0 + 20.0 * k, 0.0, 60.0), (0.7, 1.9)[k % 2]) for k in range(70)]
    sol, st, rc = S.solve(srcs, pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL))
    assert rc == pg.OK
    assert max(_residuals(S, srcs, sol.x())) <= 1.01 * RTOL


def test_resident_batch_in_several_rounds(pg):
    """Meshes that need more workgroups than the GPU has compute units run in
    rounds; with one too large for the resident form the batch runs kernel by
    kernel. A converged guess takes no iteration, a non-finite one none of the
    others' results."""
    import torch
    models = [_model(n, seed=k, f=0.4 + 0.3 * k) for k, n in enumerate([26, 4, 25, 9, 24, 22])]
    systems = [pg.System.from_model(m) for m in models]
    srcs = [m.sources[0] for m in models]
    o = pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL)
    sols, st, rc = pg.solve_many(systems, srcs, o)
    assert rc == pg.OK
    for S, src, sol in zip(systems, srcs, sols):
        assert max(_residuals(S, [src], sol.x())) <= 1.01 * RTOL
    x0 = [s.x()[0] for s in sols]
    x0[2] = torch.full_like(x0[2], float("nan"))
    sols2, st2, _ = pg.solve_many(systems, srcs, o, x0=x0)
    assert [s["iters"] > 0 for s in st2] == [False, False, True, False, False, False]
    assert [s["used_fallback"] for s in st2] == [0, 0, 1, 0, 0, 0]
    assert max(_residuals(systems[2], [srcs[2]], sols2[2].x())) <= 1.01 * RTOL
    big = _model(43)
    systems.append(pg.System.from_model(big))
    sols3, st3, rc = pg.solve_many(systems, srcs + [big.sources[0]], o)
    assert rc == pg.OK
    for S, src, sol in zip(systems, srcs + [big.sources[0]], sols3):
        assert max(_residuals(S, [src], sol.x())) <= 1.01 * RTOL


def test_resident_iteration_limit(pg):
    m = _model(8)
    S = pg.System.from_model(m)
    sol, st, rc = S.solve(m.sources, pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL, max_iter=16),
                          allow_not_converged=True)
    assert rc == pg.NOT_CONVERGED and st[0]["status"] == pg.NOT_CONVERGED and st[0]["iters"] <= 16
    sol, st, rc = S.solve(m.sources, pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL))
    assert rc == pg.OK and max(_residuals(S, m.sources, sol.x())) <= 1.01 * RTOL


# 2 and 3: one workgroup; 8: 6 workgroups (eight lanes to a sum); 12: 22;
# 21: two levels of sums; 27: two rows to a thread
@pytest.mark.parametrize("n,restart", [(2, 30), (3, 5), (8, 30), (8, 31), (8, 1), (12, 13), (21, 30), (27, 20)])
def test_resident_gmres_takes_the_steps_of_the_kernels(pg, n, restart):
    """Same cycles, same steps: the two forms differ in the order of their
    double-precision sums only, which at 1e-9 moves a cycle's last step by at
    most one. `profile` keeps the kernel-per-phase form."""
    m = _model(n, box=2000.0)
    S = pg.System.from_model(m)
    kw = dict(rtol=1e-9, restart=restart, max_iter=6000)
    sol, st, rc = S.solve(m.sources, pg.default_opts(**kw), allow_not_converged=True)
    _, stk, rck = S.solve(m.sources, pg.default_opts(profile=1, **kw), allow_not_converged=True)
    print(f"[case] gmres n={n} restart={restart} iters {st[0]['iters']} / {stk[0]['iters']}", flush=True)
    assert rc == rck and st[0]["spmv_shape"] == 1
    assert abs(st[0]["iters"] - stk[0]["iters"]) <= max(1, stk[0]["iters"] // 50)
    assert abs(st[0]["b_norm"] - stk[0]["b_norm"]) <= 1e-13 * stk[0]["b_norm"]
    res = _residuals(S, m.sources, sol.x())[0]
    if rc == pg.OK:
        assert res <= 1.01e-9
    assert abs(res - st[0]["rel_residual"]) <= 1e-12


def test_resident_gmres_several_sources_and_frequencies(pg):
    m = _model(9)
    S = pg.System.from_model(m)
    srcs = [synth.Dipole((40.0 * k, 0.0, 60.0), f) for k, f in enumerate((1.0, 0.4, 1.0))]
    sol, st, rc = S.solve(srcs, pg.default_opts(rtol=1e-9))
    assert rc == pg.OK and max(_residuals(S, srcs, sol.x())) <= 1.01e-9
    # after new conductivities the operator is formed anew
    import torch
    S.reassemble(torch.tensor(m.sigma * 1.7, device="cuda"), m.sigma_bg)
    sol, st, rc = S.solve(srcs, pg.default_opts(rtol=1e-9))
    assert rc == pg.OK and max(_residuals(S, srcs, sol.x())) <= 1.01e-9


def _small(rng):
    """One 8^3 model with a resistive plate: random plate, source, frequency and mesh jitter."""
    jit = int(rng.integers(1 << 30))
    box = ((-200.0, 200.0), (-200.0, 200.0), (-250.0 * rng.uniform(0.6, 1.6), 0.0))
    src = (float(rng.uniform(-40, 40)), 0.0, float(rng.uniform(150.0, 400.0)))
    xyz, tets = synth.kuhn_mesh(8, -1000.0, 1000.0, jit)
    c = xyz[tets].mean(axis=1)
    sig = np.ones(len(c))
    inside = np.ones(len(c), bool)
    for k in range(3):
        inside &= (c[:, k] >= box[k][0]) & (c[:, k] <= box[k][1])
    sig[inside] = float(np.exp(rng.uniform(np.log(0.005), np.log(0.05))))
    return xyz, tets, sig, src


# Model 17 of this sequence starts its third refinement step with |r^T z| a
# millionth of |r|^2 on the coarse split: its |r| wandered for 19,000
# iterations. No limit on the iterations but the one the rule implies: three
# ordinary steps (under 1,000 in all for these models), at most four stopped
# ones of a few hundred more each.
def test_resident_column_that_wanders_restarts(pg):
    print("[case] wandering column", flush=True)
    rng = np.random.default_rng([7, 11])
    models, srcs = [], []
    for _ in range(96):
        f = float(rng.uniform(0.1, 2.0))
        xyz, tets, sig, p = _small(rng)
        srcs.append(synth.Dipole(p, f))
        models.append(synth.Model("small", xyz, tets, sig, 1.0, [srcs[-1]], np.zeros((1, 3)), 8, (-1000.0, 1000.0)))
    sys = [pg.System.from_model(m) for m in models]
    o = pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=1e-12)
    sols, st, rc = pg.solve_many(sys, srcs, o)
    assert rc == pg.OK
    print(f"  iters {max(s['iters'] for s in st)}", flush=True)
    assert max(s["iters"] for s in st) < 4000
    for k in (0, 17, 95):
        assert _residuals(sys[k], [srcs[k]], sols[k].x())[0] <= 1.01e-12


# The concatenation of a batch: a mesh of one tile, one whose rows end in the
# middle of a tile, one whose entries need several blocks, and the last row
# pointer with and without padding; a system named twice.
@pytest.mark.parametrize("ns", [[2], [5, 2], [12, 2, 9], [3, 12, 3]])
def test_batch_of_unlike_systems_equals_single_solves(pg, ns):
    print(f"[case] batch {ns}", flush=True)
    ms = [_model(n, seed=11 + k) for k, n in enumerate(ns)]
    sys = [pg.System.from_model(m) for m in ms]
    srcs = [m.sources[0] for m in ms]
    sys.append(sys[0])
    srcs.append(synth.Dipole((-120.0, 40.0, 60.0), 0.7))
    o = pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL)
    sols, _, rc = pg.solve_many(sys, srcs, o)
    assert rc == pg.OK
    for k, S in enumerate(sys):
        assert _residuals(S, [srcs[k]], sols[k].x())[0] <= 1.01 * RTOL
