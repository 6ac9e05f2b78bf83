"""A plain GMRES solve that the one-launch form does not take. Marked `gpu`.

It is decided before anything is allocated or formed for that form: the first
solve does not take the two vectors that form needs beside its own more than a
profiled one, which never asks for it (allocations come in 2 MiB, less than a
vector of these meshes).
"""
import numpy as np
import pytest

from paper_1808_00186_amd import synth

pytestmark = pytest.mark.gpu


# a restart beyond the one-launch form's 31; a mesh beyond its 470,000 unknowns
@pytest.mark.parametrize("n,restart", [(30, 40), (42, 20)])
def test_a_solve_that_does_not_fit_pays_for_its_own_form_only(n, restart):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1808_00186_amd import petgem as pg
    xyz, tets = synth.kuhn_mesh(n, -5000.0, 5000.0, 3)
    sig = synth.marine_sigma(synth.centroids(xyz, tets), ((-2000, 2000), (-2000, 2000), (-1500, -1300)), 0.02)
    src = [synth.Dipole((30.0, 0.0, 50.0), 1.0)]
    print(f"[case] gmres n={n} restart={restart}", flush=True)

    def taken(profile):
        S = pg.System(xyz, tets, sig, 3.3)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        S.solve(src, pg.default_opts(rtol=1e-2, restart=restart, profile=profile))
        torch.cuda.synchronize()
        return before - torch.cuda.mem_get_info()[0], 16 * S.n_dof
    taken(1)
    (own, vector), (plain, _) = taken(1), taken(0)
    print(f"  {own} bytes, not profiled {plain}", flush=True)
    assert vector > 2 << 20 and plain < own + 2 * vector
