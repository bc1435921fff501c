"""The packet on grids of few planes: its norm is summed on one, two, four or
eight planes at a time by their number."""
import numpy as np
import pytest

import oracle
from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nz", [1, 2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("nxy", [(23, 12), (40, 37)])
def test_packet_on_few_planes(prec, nz, nxy):
    n = (*nxy, nz)
    print("packet", prec, n, flush=True)
    s = tdse.Sim(tdse.make_desc(*n, 0.2, 0.2, 0.2, precision=prec, dt_frac=0.5), pingpong=False)
    dt, _ = s.finalize()
    r0, k0, sigma = tuple(0.1 * x for x in n), (0.3, -0.2, 1.1), 1.5
    s.init_gaussian(r0, k0, sigma)
    R, I = oracle.init_gaussian(oracle.Grid(*n, 0.2, 0.2, 0.2, 1.0, 1.0), r0, k0, sigma, dt)
    # FP64: products of three factors and a norm of three sums, a few ulp of
    # the largest value; FP32: one rounding more
    tol = 1e-13 if prec == "f64" else 1.5e-7
    for got, ref in ((s.psi_r, R), (s.psi_i, I)):
        assert np.max(np.abs(got.double().cpu().numpy() - ref)) <= tol * np.max(np.abs(R))
