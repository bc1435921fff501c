"""The march loop of 1024-thread two-step tiles against the one-pass step:
chunks around the multiples of six planes it takes, detection faces at every
place of a run of six, CAP planes inside and outside it, tiles that leave
idle threads and idle wavefronts.  The cell arithmetic is the same, so
states, records and pixels are the same bits and the FP64 sums (of at most
2^17 terms in another order) agree to 1e-12 of their scale."""
import pytest
import torch

from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

# precision, extents, tile width, tile height, z chunk, CAP, k_det, z boundary
CASES = [("f32", (64, 48, 64), 64, 16, 64, 0, 40 + j, 0) for j in range(6)] + [
    ("f32", (64, 48, zc + 12), 64, 0, zc, 9, 7, 0) for zc in (6, 7, 8, 13, 14, 19)] + [
    ("f64", (32, 40, 40), 32, 16, zc, 6, 21, 0) for zc in (40, 20, 17)] + [
    ("f32", (40, 30, 45), 40, 22, 45, 22, 44, 1),
    ("f32", (38, 30, 45), 38, 12, 23, 5, 0, 0),
    ("f32", (37, 29, 53), 16, 9, 27, 6, 30, 0),
    ("f64", (37, 29, 53), 16, 20, 53, 6, 52, 1),
]


@pytest.mark.parametrize("prec,n,tx,ty,zc,cap,kdet,bcz", CASES)
def test_march_is_bitwise_the_one_pass_step(prec, n, tx, ty, zc, cap, kdet, bcz):
    print("march", prec, n, tx, ty, zc, cap, kdet, bcz, flush=True)
    h, steps = 6, 26

    def run(**tile):
        d = tdse.make_desc(*n, 0.2, 0.21, 0.22, 0.6582119569, 0.0568563, precision=prec, bc=(0, 0, bcz),
                           k_det=kdet, record_every=h, max_records=steps // h + 1,
                           flags=tdse.FLAG_PIXEL_INTEGRAL)
        s = tdse.Sim(d)
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        r = [torch.rand((n[2], n[1], n[0]), generator=g, device="cuda", dtype=torch.float64)
             for _ in range(3)]
        s.v.copy_(-30.0 * r[0])
        if cap:
            s.set_cap_quadratic(cap, cap, 50.0)
        s.finalize()
        s.set_state(r[1] - 0.5, r[2] - 0.5, step=0)
        s.set_tile(fused=1, **tile)
        s.step(steps)
        return s, s.detect()

    one, a = run(two_step=0)
    two, b = run(two_step=1, two_step_tx=tx, two_step_rows=1, two_step_threads=1024, two_step_zc=zc,
                 two_step_ty=ty, two_step_prefetch=1)
    assert torch.equal(two.psi_r, one.psi_r) and torch.equal(two.psi_i, one.psi_i)
    assert torch.equal(two.records, one.records) and torch.equal(two.pixel, one.pixel)
    scale = one.scalars.abs().max()
    assert float((two.scalars - one.scalars).abs().max() / scale) < 1e-12
    assert b.flux == pytest.approx(a.flux, rel=1e-12, abs=1e-12 * float(scale))


@pytest.mark.parametrize("prec,n,bc,one_round", [
    ("f32", (144, 144, 288), (0, 0, 0), True),
    ("f32", (200, 180, 300), (0, 0, 1), True),
    ("f64", (160, 160, 160), (0, 0, 0), True),
    ("f32", (160, 160, 160), (0, 0, 0), False),     # below 5 Mi cells
    ("f32", (144, 144, 288), (1, 0, 0), False),     # no march with a zero boundary in x
])
def test_default_tile_of_mid_size_grids(prec, n, bc, one_round):
    """From 5 Mi cells (FP64: 4 M) on, the default is a 1024-thread tile in
    one round of the CUs; its states and records are the one-pass step's."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule's tiles are those of a 256-CU device")
    print("mid-size default", prec, n, bc, flush=True)
    out = []
    for force_one in (False, True):
        d = tdse.make_desc(*n, 0.2, 0.21, 0.22, 0.6582119569, 0.0568563, precision=prec, bc=bc,
                           k_det=n[2] // 2, record_every=10, max_records=3)
        s = tdse.Sim(d)
        g = torch.Generator(device="cuda")
        g.manual_seed(9)
        r = [torch.rand((n[2], n[1], n[0]), generator=g, device="cuda") for _ in range(3)]
        s.v.copy_(-30.0 * r[0])
        s.set_cap_quadratic(10, 10, 50.0)
        s.finalize()
        s.set_state(r[1] - 0.5, r[2] - 0.5, step=0)
        t = s.get_tile()
        if force_one:
            s.set_tile(fused=1, two_step=0, fused_prefetch=1)
        else:
            assert (t.two_step == 1 and t.two_step_threads == 1024 and t.two_step_zc < 32) == one_round
        s.step(21)
        out.append(s)
    a, b = out
    assert torch.equal(a.psi_r, b.psi_r) and torch.equal(a.psi_i, b.psi_i) and torch.equal(a.records, b.records)
