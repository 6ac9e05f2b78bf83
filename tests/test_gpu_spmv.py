"""The product with A on vectors that overlap its result. Marked `gpu`.

The same kernel forms both results, so they are the same bits.
"""
import ctypes as C

import numpy as np
import pytest

from paper_1808_00186_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def system():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1808_00186_amd import petgem
    xyz, tets = synth.kuhn_mesh(14, -1000.0, 1000.0, 3)
    return petgem.System(xyz, tets, np.where(xyz[tets].mean(axis=1)[:, 2] > 0, 3.3, 1.0), 3.3)


# y at this many elements from x, as a part of n: in place, shifted either way
# by one element, by half, side by side
@pytest.mark.parametrize("num,den,plus", [(0, 1, 0), (0, 1, 1), (0, 1, -1), (1, 2, 0), (-1, 2, 0), (1, 1, 0), (-1, 1, 0)])
def test_product_of_overlapping_vectors(system, num, den, plus):
    import torch
    from paper_1808_00186_amd import petgem as pg
    n = system.n_dof
    shift = num * n // den + plus
    print(f"[case] spmv n={n} shift={shift}", flush=True)
    rng = np.random.default_rng(5)
    x = torch.tensor(rng.normal(size=(n, 2)), device="cuda").view(torch.complex128).reshape(n)
    want = system.spmv(0.7, x)
    buf = torch.zeros(3 * n, dtype=torch.complex128, device="cuda")
    for _ in range(2):
        buf[n:2 * n] = x
        base = buf.data_ptr()
        rc = pg.lib().petgem_spmv(system.handle, 0.7, C.c_void_p(base + 16 * n), C.c_void_p(base + 16 * (n + shift)),
                                  pg._stream())
        assert rc == pg.OK
        assert torch.equal(torch.view_as_real(buf[n + shift:2 * n + shift]), torch.view_as_real(want))
        if abs(shift) >= n:
            assert torch.equal(torch.view_as_real(buf[n:2 * n]), torch.view_as_real(x))
