"""Steps of a GMRES cycle that brings its residual far down, against GMRES with a
basis orthogonal to rounding (every step orthogonalised twice, in numpy).
Marked `gpu`.

The residual's estimate ends the cycle; with an orthogonal basis it follows
the residual, so the steps are those of the reference, give or take the last one.
A change of the source's place by a nanometre changes the roundings.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import fem
from paper_1808_00186_amd import synth

pytestmark = pytest.mark.gpu


def _steps(A, b, m, rtol):
    """Total steps of right-Jacobi GMRES(m)."""
    Ah = (A @ sp.diags(1.0 / A.diagonal())).tocsr()
    x, tol, total = np.zeros_like(b), rtol * np.linalg.norm(b), 0
    while True:
        r = b - Ah @ x
        rn = np.linalg.norm(r)
        if rn <= tol:
            return total
        V, H = [r / rn], np.zeros((m + 1, m), complex)
        for j in range(m):
            w = Ah @ V[j]
            for _ in range(2):
                c = np.array([np.vdot(v, w) for v in V])
                H[:j + 1, j] += c
                w = w - sum(ci * v for ci, v in zip(c, V))
            H[j + 1, j] = np.linalg.norm(w)
            V.append(w / H[j + 1, j])
            e = np.zeros(j + 2, complex)
            e[0] = rn
            y = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[0]
            if np.linalg.norm(e - H[:j + 2, :j + 1] @ y) <= tol:
                break
        x = x + sum(yi * v for yi, v in zip(y, V))
        total += j + 1


# 26 unknowns in one cycle, in one launch and kernel by kernel (profile); 3,000
# unknowns with a restart that only the kernels take
@pytest.mark.parametrize("n,box,restart,forms", [(2, 2000.0, 30, (0, 1)), (8, 5000.0, 60, (0,))])
def test_steps_of_a_deep_cycle(n, box, restart, forms):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1808_00186_amd import petgem as pg
    xyz, tets = synth.kuhn_mesh(n, -box, box, 5 + n)
    sig = synth.marine_sigma(synth.centroids(xyz, tets), ((-0.4 * box, 0.4 * box), (-0.4 * box, 0.4 * box),
                                                          (-0.6 * box, -0.2 * box)), 0.02)
    sys, S = fem.assemble(xyz, tets, sig), pg.System(xyz, tets, sig, 3.3)
    A = fem.system_matrix(sys, 1.0).tocsr()
    for k in range(6):
        d = synth.Dipole((30.0 + 1e-9 * k, 0.0, 50.0), 1.0)
        b = fem.rhs(xyz, tets, sig, 3.3, sys.topo, d.pos, d.dir, d.freq)
        want = _steps(A, b, restart, 1e-9)
        got = []
        for profile in forms:
            _, st, rc = S.solve([d], pg.default_opts(rtol=1e-9, restart=restart, profile=profile))
            assert rc == pg.OK
            got.append(st[0]["iters"])
        print(f"[case] gmres n={n} restart={restart} draw {k}: {got}, orthogonal {want}", flush=True)
        assert all(abs(g - want) <= 1 for g in got)
