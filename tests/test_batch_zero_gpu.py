"""A batch of 1024-thread two-step tiles in which one member has a zero x
boundary: the launch then takes the instance without the march loop for all
of them, and each member is still what it is alone, bit for bit."""
import pytest
import torch

from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

MEMBERS = [((64, 48, 70), (0, 0, 0), 9), ((48, 40, 50), (1, 0, 0), 0), ((40, 64, 45), (0, 0, 1), 6),
           ((56, 33, 40), (0, 1, 0), 6)]
H, STEPS = 10, 50


def desc(prec, n, bc):
    return tdse.make_desc(*n, 0.2, 0.21, 0.22, 0.6582119569, 0.0568563, precision=prec, bc=bc, k_det=n[2] // 2,
                          record_every=H, max_records=STEPS // H + 1)


def set_up(s, i, n, cap):
    g = torch.Generator(device="cuda")
    g.manual_seed(20 + i)
    r = [torch.rand((n[2], n[1], n[0]), generator=g, device="cuda", dtype=torch.float64) for _ in range(3)]
    s.v.copy_(-30.0 * r[0])
    torch.cuda.synchronize()
    if cap:
        s.set_cap_quadratic(cap, cap, 50.0)
    s.finalize()
    s.set_state(r[1] - 0.5, r[2] - 0.5, step=0)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("which", [(0, 1), (0, 2), (0, 1, 2, 3)])
def test_mixed_boundaries_equal_single_runs(prec, which):
    print("mixed batch", prec, which, flush=True)
    ms = [MEMBERS[i] for i in which]
    b = tdse.Batch([desc(prec, n, bc) for n, bc, _ in ms])
    for i, (m, (n, _, cap)) in enumerate(zip(b.members, ms)):
        set_up(m, i, n, cap)
    b.set_two_step(True, tx=16, zc=25, prefetch=True, rows=1, threads=1024)
    b.prepare()
    b.run(STEPS)
    torch.cuda.synchronize()
    assert all(st == tdse.OK for st in b.status())
    for i, (m, (n, bc, cap)) in enumerate(zip(b.members, ms)):
        one = tdse.Sim(desc(prec, n, bc))
        set_up(one, i, n, cap)
        one.set_tile(fused=1, two_step=0, fused_prefetch=1)
        one.step(STEPS)
        assert torch.equal(m.psi_r, one.psi_r) and torch.equal(m.psi_i, one.psi_i)
        assert torch.equal(m.records, one.records)
        # sums of at most 2^18 terms in another order
        scale = float(one.scalars.abs().max())
        assert float((m.scalars - one.scalars).abs().max()) <= 1e-12 * scale
