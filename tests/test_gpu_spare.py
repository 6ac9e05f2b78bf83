"""Solves and right-hand sides without room for what only makes them faster.
Marked `gpu`.

The limit takes the place of a device without memory: both end in the same
failed allocation. At every limit, from none of it up to all, the forms that do
without must give the results: the true residual within its tolerance (1 % for the
rounding of its own evaluation), right-hand sides the same bits.
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
    return synth.Model(f"spare-{n}", xyz, tets, sig, 3.3, [synth.Dipole((30.0, 0.0, 50.0), 1.0)], np.zeros((1, 3)), n,
                       (-3000.0, 3000.0))


def _sources(cols):
    return [synth.Dipole((-200.0 + 90.0 * k, 10.0, 50.0), (0.5, 1.3, 2.0)[k % 3]) for k in range(cols)]


def _residual(S, src, x):
    b = S.rhs([src])[0]
    return float((b - S.spmv(src.freq, x.contiguous())).norm() / b.norm())


def _solve(pg, systems, what):
    """One pass; the residuals of its solutions."""
    if what == "batch":
        srcs = _sources(len(systems))
        sols, _, rc = pg.solve_many(systems, srcs, pg.default_opts(method=pg.COCG, precision=pg.MIXED, rtol=RTOL))
        assert rc == pg.OK
        return [(S, d, sol.x()[0]) for S, d, sol in zip(systems, srcs, sols)]
    srcs = _sources(what[1])
    o = pg.default_opts(rtol=RTOL, restart=30) if what[0] == "gmres" else pg.default_opts(
        method=pg.COCG, precision=pg.MIXED, rtol=RTOL)
    sol, _, rc = systems[0].solve(srcs, o)
    assert rc == pg.OK
    return [(systems[0], d, x) for d, x in zip(srcs, sol.x())]


@pytest.mark.parametrize("what,ns", [(("gmres", 2), [9]), (("cocg", 1), [12]), (("cocg", 9), [9]), ("batch", [9, 5, 12])])
def test_solves_at_every_limit(pg, what, ns):
    models = [_model(n) for n in ns]

    def check(systems):
        out = _solve(pg, systems, what)
        held = [S.spare_bytes() for S in systems]
        for S, d, x in out:
            S.set_spare_limit(0)      # the check's own right-hand side takes none
            assert _residual(S, d, x) <= 1.01 * RTOL
        return held
    need = check([pg.System.from_model(m) for m in models])
    assert all(b > 0 for b in need)
    print(f"[case] {what} {ns}: needs {need}", flush=True)
    for part in (0.0, 0.05, 0.3, 0.6, 0.9, 1.0):
        systems = [pg.System.from_model(m) for m in models]
        limits = [int(part * b) for b in need]
        for S, lim in zip(systems, limits):
            S.set_spare_limit(lim)
        held = check(systems)
        print(f"  {part}: holds {held}", flush=True)
        assert all(h <= lim for h, lim in zip(held, limits))
        if part == 1.0:
            assert held == need
        # with room again the one-launch form comes back
        for S in systems:
            S.set_spare_limit(-1)
            assert S.spare_bytes() == 0
        assert check(systems) == need
    # one mesh of a batch without room: all by kernels, and none holds what it cannot use
    if what == "batch":
        systems = [pg.System.from_model(m) for m in models]
        systems[-1].set_spare_limit(1000)
        _solve(pg, systems, what)
        assert [S.spare_bytes() for S in systems] == [0, 0, 0]


@pytest.mark.parametrize("layered", [False, True])
def test_right_hand_sides_at_every_limit(pg, layered):
    m = synth.layered_marine() if layered else _model(9)
    srcs = [synth.Dipole((-100.0 + 30.0 * k, 10.0, 60.0), 0.5 + 0.1 * k) for k in range(5)]
    S = pg.System.from_model(m)
    want = S.rhs(srcs).cpu().numpy()
    need = S.spare_bytes()
    print(f"[case] rhs layered={layered}: needs {need}", flush=True)
    assert need > 0
    for lim in (0, need - 1, need, -1):
        S.set_spare_limit(lim)
        assert S.spare_bytes() == 0
        assert np.array_equal(S.rhs(srcs).cpu().numpy(), want)
        assert S.spare_bytes() == (need if lim in (need, -1) else 0)
        assert np.array_equal(S.rhs(srcs[:1]).cpu().numpy(), want[:1])


def test_limit_arguments(pg):
    S = pg.System.from_model(_model(4))
    with pytest.raises(pg.PetgemError) as e:
        S.set_spare_limit(-2)
    assert e.value.code == pg.INVALID_ARG
    assert pg.lib().petgem_spare_bytes(None) == -1
    assert pg.lib().petgem_set_spare_limit(None, 0) == pg.INVALID_ARG
