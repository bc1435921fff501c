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
