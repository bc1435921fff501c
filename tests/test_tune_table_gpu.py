"""The measured tiles against the library's defaults: on grids that step on
bricks by default, an entry with one-pass fields of its own would take them
off the bricks (128x128x256 FP32 20 -> 26 us a step)."""
import pytest

from paper_2401_07416_amd import tdse, tuning, workloads

pytestmark = pytest.mark.gpu

SMALL = [(prec, w) for w in (workloads.c1_free_gaussian(), workloads.c2_reduced(), workloads.c5_adjoint())
         for prec in ("f32", "f64")]


@pytest.mark.parametrize("prec,w", SMALL)
def test_table_keeps_small_grids_on_their_default_steps(prec, w):
    print("table", prec, w.nx, w.ny, w.nz, flush=True)
    counts = []
    for tile in (None, tuning.tile_for(w, prec)):
        s = tdse.sim_from_workload(w, precision=prec, steps=40)
        if tile is not None:
            s.set_tile(**tile)
        s.set_timing(True)
        s.step(8)
        counts.append({k: v[1] for k, v in s.timing_read().items()})
    assert counts[0] == counts[1]
