"""Runs on bricks cut into calls of every kind: a call of one step runs as two
half-steps in place, and the state, the records and the sums are those of one
call over the same steps, bit for bit."""
import pytest
import torch

from tests.test_brick_gpu import CASES, start

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,bc", CASES)
def test_single_steps_are_bitwise_one_run(prec, n, bc):
    h, steps = 7, 16
    print("single steps on bricks", prec, n, bc, flush=True)
    whole = start(prec, n, bc, h, steps)
    whole.step(steps)
    single = start(prec, n, bc, h, steps)
    single.set_timing(True)
    for _ in range(steps):
        single.step(1)
    t = single.timing_read()
    # two launches a step, no second state pair to copy back from
    assert {k: v[1] for k, v in t.items()} == {"half_i": steps, "half_r": steps, "fused": 0, "two_step": 0}
    a, b = whole.detect(), single.detect()
    for x, y in ((whole.psi_r, single.psi_r), (whole.psi_i, single.psi_i), (whole.records, single.records),
                 (whole.pixel, single.pixel), (whole.scalars, single.scalars)):
        assert torch.equal(x, y)
    assert a.flux == b.flux and a.step == b.step == steps


def launches(s):
    """Launches by kind since the last read: plain ones, then those with a record."""
    t = s.timing_read_split()
    kinds = ("half_i", "half_r", "fused", "two_step")
    return tuple(t[k][1] for k in kinds), tuple(t[k + "_rec"][1] for k in kinds)


@pytest.mark.parametrize("n,h", [((96, 96, 192), 10), ((80, 80, 160), 7), ((128, 128, 128), 3)])
def test_grids_of_several_rounds_pair_only_steps_without_a_record(n, h):
    """More bricks than the chip holds: pairs without a record on bricks, the
    steps beside them on the one-pass kernel, the states and records its own."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule's line is that of a 256-CU device")
    print("several rounds of bricks", n, h, flush=True)
    steps = 4 * h
    one = start("f32", n, (0, 0, 0), h, steps)
    one.set_tile(two_step=0, fused_prefetch=1)
    one.step(steps)
    s = start("f32", n, (0, 0, 0), h, steps)
    s.set_timing(True)
    s.step(steps)
    pairs = (h - 1) // 2
    assert launches(s) == ((0, 0, 4 * (h - 1 - 2 * pairs), 4 * pairs), (0, 0, 4, 0))
    split = start("f32", n, (0, 0, 0), h, steps)
    split.set_timing(True)
    split.step(1)
    assert launches(split)[0] == (1, 1, 0, 0)
    split.step(2)
    a, b = launches(split)
    assert a[3] == b[3] == 0        # two one-pass steps, not two on bricks
    split.step(steps - 3)
    for x in (s, split):
        assert torch.equal(x.psi_r, one.psi_r) and torch.equal(x.psi_i, one.psi_i)
        assert torch.equal(x.records, one.records) and torch.equal(x.pixel, one.pixel)
        # sums of at most 2^21 terms in another order
        scale = float(one.scalars.abs().max())
        assert float((x.scalars - one.scalars).abs().max()) <= 1e-12 * scale


@pytest.mark.parametrize("n,h,pairs", [((128, 128, 128), 1, 0), ((128, 128, 128), 2, 0), ((66, 64, 64), 3, 0),
                                       ((66, 64, 64), 4, 6), ((64, 64, 64), 1, 0), ((64, 64, 64), 2, 6)])
def test_short_record_intervals(n, h, pairs):
    """Where a record costs the bricks more than they save, none are taken."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule's line is that of a 256-CU device")
    print("records every", h, n, flush=True)
    s = start("f32", n, (0, 0, 0), h, 12)
    s.set_timing(True)
    s.step(12)
    plain, rec = launches(s)
    assert plain[3] + rec[3] == pairs and plain[2] + rec[2] == 12 - 2 * pairs
