"""tdse_autotune on a mid-size grid finds the library's default two-step tile
again, its height included, from a handle whose tile was changed before
(192x192x384 FP32: 36.5 us a step, 48 and more on the other candidates)."""
import pytest
import torch

from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

FIELDS = ("two_step", "two_step_tx", "two_step_rows", "two_step_threads", "two_step_zc", "two_step_ty")


def test_autotune_finds_the_default_tile_with_its_height():
    print("autotune 192x192x384", flush=True)
    s = tdse.Sim(tdse.make_desc(192, 192, 384, 0.2, 0.2, 0.2, 0.6582119569, 0.0568563, precision="f32"))
    s.finalize()
    t = s.get_tile()
    want = [getattr(t, f) for f in FIELDS]
    assert t.two_step == 1 and t.two_step_threads == 1024 and t.two_step_ty > 0
    # another tile, of another height
    s.set_tile(two_step=1, two_step_tx=48, two_step_rows=1, two_step_threads=512, two_step_zc=32,
               two_step_ty=want[-1] - 7)
    s.set_state(torch.zeros_like(s.psi_r), torch.zeros_like(s.psi_i))
    t = s.autotune(steps=20, flags=4)
    assert [getattr(t, f) for f in FIELDS] == want
