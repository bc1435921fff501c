"""The atom-sum potential kernel against the oracle where its tiles and
candidate lists can go wrong: partial tiles, boxes shorter than the cutoff
and than twice the cutoff plus a tile (several images of an atom near one
tile), zero boundaries, atoms outside the box and far from it, more
candidates than one pass of a workgroup keeps, none at all."""
import numpy as np
import pytest

import oracle
from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

CASES = [
    ((33, 9, 17), (0, 0, 0), 2.0, 40, 1.0),
    ((37, 29, 53), (1, 0, 0), 6.0, 60, 1.0),
    ((37, 29, 53), (0, 1, 1), 6.0, 60, 1.5),
    ((96, 65, 80), (0, 0, 0), 3.0, 700, 1.0),
    ((16, 12, 40), (0, 0, 0), 6.0, 30, 3.0),
    ((8, 8, 8), (0, 0, 0), 50.0, 3, 1.0),
    ((40, 24, 31), (0, 0, 0), 1.1, 25, 1e8),
    ((40, 24, 31), (0, 0, 1), 1.1, 0, 1.0),
]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,bc,cutoff,atoms,spread", CASES)
def test_potential_matches_oracle(prec, n, bc, cutoff, atoms, spread):
    print("potential", prec, n, bc, cutoff, atoms, spread, flush=True)
    rng = np.random.default_rng(3)
    L = 0.2 * np.array(n)
    a = np.zeros((atoms, 5))
    a[:, :3] = L * (0.5 + spread * rng.uniform(-0.5, 0.5, (atoms, 3)))
    a[:, 3] = rng.choice([1.0, 6.0, 14.0], atoms)
    a[:, 4] = rng.uniform(0.5, 1.5, atoms)
    if spread > 1e6:
        a[:5, :3] = L * rng.uniform(0.0, 1.0, (5, 3))   # among those far out
    s = tdse.Sim(tdse.make_desc(*n, 0.2, 0.2, 0.2, precision=prec, bc=bc), pingpong=False)
    s.build_potential(a, cutoff=cutoff)
    v = s.v.double().cpu().numpy()
    ref = oracle.potential(oracle.Grid(*n, 0.2, 0.2, 0.2, 1.0, 1.0, bc=bc), a, soft=0.1, cutoff=cutoff,
                           kappa=14.3996454784, a0=0.529177210903, screened=True)
    # FP64: at most `atoms` terms of one sign, a few ulp each; FP32: one rounding more
    tol = 1e-14 * max(atoms, 10) if prec == "f64" else 1e-7
    assert np.max(np.abs(v - ref)) <= tol * max(np.max(np.abs(ref)), 1e-300)
