"""Which solves run in one launch, and what happens when a wait of theirs runs
out. Marked `gpu`.

With a limit of one poll a wait gives up as soon as another workgroup is not
there yet; the kernel then ends by itself and the solve runs again kernel by
kernel. Its results are held to the true residual (1 % for the rounding of its own
evaluation).
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


def _model(n, seed=5):
    xyz, tets = synth.kuhn_mesh(n, -3000.0, 3000.0, seed + n)
    sig = synth.marine_sigma(synth.centroids(xyz, tets), ((-1200, 1200), (-1200, 1200), (-1800, -600)), 0.02)
    return synth.Model(f"wait-{n}", xyz, tets, sig, 3.3, [synth.Dipole((30.0, 0.0, 50.0), 1.0)], np.zeros((1, 3)), n,
                       (-3000.0, 3000.0))


def _sources(cols):
    return [synth.Dipole((-200.0 + 90.0 * k, 10.0, 50.0), (0.5, 1.3, 2.0)[k % 3]) for k in range(cols)]


def _opts(pg, form, **kw):
    if form == "gmres":
        return pg.default_opts(rtol=RTOL, **kw)
    return pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL, **kw)


def _check(S, srcs, xs):
    b = S.rhs(srcs)
    for k, (d, x) in enumerate(zip(srcs, xs)):
        assert float((b[k] - S.spmv(d.freq, x.contiguous())).norm() / b[k].norm()) <= 1.01 * RTOL


# 9: 8 workgroups, one level of sums; 22: 139, two levels
@pytest.mark.parametrize("form,cols,n", [("gmres", 1, 9), ("gmres", 2, 16), ("cocg", 1, 9), ("cocg", 1, 22), ("cocg", 9, 9)])
def test_a_wait_that_runs_out(pg, form, cols, n):
    print(f"[case] wait {form} cols={cols} n={n}", flush=True)
    S, srcs = pg.System.from_model(_model(n)), _sources(cols)

    def solve():
        sol, st, rc = S.solve(srcs, _opts(pg, form))
        assert rc == pg.OK
        _check(S, srcs, sol.x())
        return [s["one_launch"] for s in st]
    assert solve() == [1] * cols
    S.set_wait_limit(1)
    got = solve()
    # a GMRES source after the one whose wait ran out does not try
    assert got == ([2] + [0] * (cols - 1) if form == "gmres" else [2] * cols)
    assert solve() == [0] * cols          # nor does the next solve
    S.set_wait_limit(0)
    assert solve() == [1] * cols


def test_a_wait_that_runs_out_in_a_batch(pg):
    print("[case] wait batch", flush=True)
    systems = [pg.System.from_model(_model(n)) for n in (9, 4, 14)]
    srcs = _sources(3)

    def solve(x0=None):
        sols, st, rc = pg.solve_many(systems, srcs, _opts(pg, "cocg"), x0=x0)
        assert rc == pg.OK
        for S, d, sol in zip(systems, srcs, sols):
            _check(S, [d], sol.x())
        return [s["one_launch"] for s in st], [sol.x()[0] for sol in sols]
    form, x = solve()
    assert form == [1, 1, 1]
    systems[0].set_wait_limit(1)
    # a guess is taken again by the second try: the first mesh has none, the others' is rough
    assert solve([None, 0.9 * x[1], 0.5 * x[2]])[0] == [2, 2, 2]
    assert solve()[0] == [0, 0, 0]
    systems[0].set_wait_limit(0)
    assert solve()[0] == [1, 1, 1]


def test_which_solves_run_in_one_launch(pg):
    print("[case] which form", flush=True)

    def form(S, **kw):
        f = kw.pop("form", "cocg")
        _, st, _ = S.solve(_sources(kw.pop("cols", 1)), _opts(pg, f, **kw), allow_not_converged=True)
        return {s["one_launch"] for s in st}
    S = pg.System.from_model(_model(8))
    assert form(S) == form(S, cols=3) == form(S, form="gmres") == form(S, form="gmres", restart=31) == {1}
    for kw in (dict(profile=1), dict(spmm_shape=40104), dict(precond=pg.SSOR), dict(form="gmres", restart=32),
               dict(form="gmres", profile=1)):
        assert form(S, **kw) == {0}, kw
    # 546,000 unknowns: too many rows for the compute units' registers
    big = pg.System.from_model(_model(43))
    assert form(big, max_iter=20) == form(big, form="gmres", max_iter=30) == {0}
    _, st, _ = pg.solve_many([S, big], _sources(2), _opts(pg, "cocg", max_iter=20), allow_not_converged=True)
    assert [s["one_launch"] for s in st] == [0, 0]
    with pytest.raises(pg.PetgemError):
        S.set_wait_limit(-1)
