"""The set-up passes around the potential at the sizes where they can go
wrong: the packet's writer at every vector width and in partial plane chunks,
the range of V with cells past the last whole vector and non-finite values
anywhere."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

SHAPES = [(64, 33, 50), (66, 7, 129), (37, 29, 53), (4, 4, 1), (1, 1, 5), (2, 3, 4)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", SHAPES)
def test_packet_matches_oracle(prec, n):
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


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", SHAPES + [(130, 70, 90)])
def test_range_of_v(prec, n):
    print("range of V", prec, n, flush=True)
    s = tdse.Sim(tdse.make_desc(*n, 0.2, 0.2, 0.2, precision=prec, dt_frac=0.5), pingpong=False)
    cells = s.v.numel()
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    flat = s.v.view(-1)
    for where in {0, cells // 2, cells - 1}:
        flat.copy_(-5.0 * torch.rand(cells, generator=g, device="cuda", dtype=torch.float64))
        flat[where] = -7.25
        if cells > 1:
            flat[(where + 1) % cells] = 3.5
        e_max, _ = tdse.time_step_bound(s.desc, -7.25, max(3.5 if cells > 1 else -7.25, float(flat.max())))
        assert s.finalize()[1] == e_max
        for bad in (float("nan"), float("inf"), -float("inf")):
            flat[where] = bad
            with pytest.raises(tdse.TdseError) as e:
                s.finalize()
            assert e.value.status == tdse.ERR_NONFINITE
