"""Atoms many millions of periods outside a periodic box, where the rounding
of the coordinates is larger than the slack of the tile tests: every cell
within the cutoff by the plain formula is still counted."""
import numpy as np
import pytest

import oracle
from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

# the first cell of a 32-wide tile lies just inside the cutoff of the atom,
# the tile's centre, rounded on its own, just beyond it
FAR = (445769417614.977, 3.0, 1.2000000000000002)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("axes", [(0, 1, 2), (1, 2, 0), (2, 0, 1)])
def test_far_atom_matches_oracle(prec, axes):
    print("far atom", prec, axes, flush=True)
    n = np.array((40, 24, 31))[list(axes)]
    a = np.zeros((2, 5))
    a[0, :3] = np.array(FAR)[list(axes)]
    a[1, :3] = 0.1 * n                      # and one inside the box
    a[:, 3:] = (14.0, 1.0)
    s = tdse.Sim(tdse.make_desc(*[int(x) for x in n], 0.2, 0.2, 0.2, precision=prec), pingpong=False)
    s.build_potential(a, cutoff=0.777)
    v = s.v.double().cpu().numpy()
    ref = oracle.potential(oracle.Grid(*[int(x) for x in n], 0.2, 0.2, 0.2, 1.0, 1.0), a, soft=0.1, cutoff=0.777,
                           kappa=14.3996454784, a0=0.529177210903, screened=True)
    # FP64: two terms, a few ulp each; FP32: one rounding more
    tol = 1e-13 if prec == "f64" else 1e-7
    assert np.max(np.abs(v - ref)) <= tol * np.max(np.abs(ref))
