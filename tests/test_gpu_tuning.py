"""The tuner's choice after solves and products that do without it. Marked `gpu`."""
import numpy as np
import pytest

from paper_1808_00186_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", ["gmres in one launch", "gmres by kernels", "product"])
def test_the_choice_is_there_when_it_is_asked_for(first):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1808_00186_amd import petgem as pg
    m = synth.config1()
    S = pg.System.from_model(m)
    assert S.tuning()["spmv_group"] == 0
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        S.reassemble(torch.tensor(m.sigma * 1.3, device="cuda"), m.sigma_bg)
        if first == "product":
            x = torch.ones(S.n_dof, dtype=torch.complex128, device="cuda")
            y = S.spmv(0.7, x)
        else:
            sol, st, _ = S.solve(m.sources, pg.default_opts(restart=30 if "one" in first else 40))
            assert st[0]["one_launch"] == ("one" in first)
            y = sol.x()
        t = S.tuning()
    assert t["spmv_group"] in (4, 8, 16) and S.tuning() == t
    assert min(t["spmv_ms_g4_g8_g16"]) > 0.0
    # and nothing else changes
    with torch.cuda.stream(side):
        again = S.spmv(0.7, x) if first == "product" else S.solve(
            m.sources, pg.default_opts(restart=30 if "one" in first else 40))[0].x()
    assert torch.equal(torch.view_as_real(y), torch.view_as_real(again))
