"""Steps on bricks (small grids on their default tile) against the one-pass
kernel: the same cell arithmetic, so states and records bit for bit, and the
FP64 sums to rounding; the sums of a run do not depend on how calls split
it."""
import pytest
import torch

from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

# every built shape (precision, vector width), extents that leave partial
# bricks on each axis, the smallest extents taken, zero boundaries
CASES = [
    ("f32", (64, 64, 128), (0, 0, 0)),   # W 4, 32 x 8
    ("f32", (80, 80, 80), (0, 0, 0)),    # 16 x 16
    ("f32", (96, 96, 96), (0, 1, 0)),    # 32 x 16
    ("f32", (36, 44, 30), (0, 0, 0)),    # 16 x 8
    ("f32", (66, 64, 64), (1, 0, 0)),    # W 2, 16 x 8
    ("f32", (38, 30, 50), (0, 0, 1)),    # 8 x 8
    ("f32", (37, 29, 53), (1, 1, 1)),    # W 1
    ("f64", (64, 64, 64), (0, 0, 0)),    # W 2, 16 x 8
    ("f64", (34, 22, 41), (0, 0, 1)),    # 8 x 8
    ("f64", (37, 29, 53), (1, 0, 0)),    # W 1
    ("f64", (4, 9, 12), (0, 0, 0)),
    ("f32", (4, 4, 4), (0, 0, 0)),
    ("f32", (5, 7, 11), (0, 1, 0)),
]


def start(prec, n, bc, h, steps):
    d = tdse.make_desc(*n, 0.2, 0.21, 0.22, 0.6582119569, 0.0568563, precision=prec, bc=bc,
                       k_det=n[2] - 1 if bc[2] else n[2] // 2, record_every=h,
                       max_records=steps // h + 1, flags=tdse.FLAG_PIXEL_INTEGRAL)
    s = tdse.Sim(d)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)

    def rand():
        return torch.rand((n[2], n[1], n[0]), generator=g, device="cuda", dtype=torch.float64)
    s.v.copy_(-30.0 * rand())
    cap = min(6, n[2] // 4)
    s.set_cap_quadratic(cap, cap, 50.0)
    s.finalize()
    s.set_state(rand() - 0.5, rand() - 0.5, step=0)
    return s


@pytest.mark.parametrize("prec,n,bc", CASES)
def test_bricks_are_bitwise_the_one_pass_step(prec, n, bc):
    h, steps = 7, 43
    print("bricks", prec, n, bc, flush=True)
    one = start(prec, n, bc, h, steps)
    t = one.get_tile()
    # the same tile with the prefetch flag turned asks for the one-pass kernel
    one.set_tile(two_step=0, fused_prefetch=1)
    brick = start(prec, n, bc, h, steps)
    brick.set_timing(True)
    brick.step(steps)
    assert t.two_step == 0 and brick.timing_read()["two_step"][1] > 0
    one.step(steps)
    split = start(prec, n, bc, h, steps)
    for k in (1, 2, 11, 28, 1):
        split.step(k)
    a, b, c = one.detect(), brick.detect(), split.detect()
    for s in (brick, split):
        assert torch.equal(s.psi_r, one.psi_r) and torch.equal(s.psi_i, one.psi_i)
        assert torch.equal(s.records, one.records) and torch.equal(s.pixel, one.pixel)
        # sums of at most 2^19 terms in another order
        scale = one.scalars.abs().max()
        assert float((s.scalars - one.scalars).abs().max() / scale) <= 1e-12
    assert abs(b.flux - a.flux) <= 1e-12 * float(one.scalars.abs().max())
    assert torch.equal(split.scalars, brick.scalars) and c.flux == b.flux
