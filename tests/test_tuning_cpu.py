"""tuning.autotune times the tile in force with its list, complete: the
sweep's height, which set_tile would otherwise reset, and the one-pass fields,
which the candidates before it have changed."""
import itertools
import types

import torch

from paper_2401_07416_amd import tuning


def test_autotune_times_the_tile_in_force(monkeypatch):
    clock = itertools.count(1)

    class Event:
        def __init__(self, enable_timing=False):
            pass

        def record(self):
            pass

        def synchronize(self):
            pass

        def elapsed_time(self, other):
            return float(next(clock))

    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    monkeypatch.setattr(torch.cuda, "Event", Event)
    tile = types.SimpleNamespace(fused=1, fused_rows=2, fused_zc=4, fused_prefetch=0, fused_threads=256,
                                 two_step=1, two_step_tx=96, two_step_rows=1, two_step_zc=24,
                                 two_step_prefetch=1, two_step_threads=1024, two_step_ty=24)
    timed = []
    sim = types.SimpleNamespace(get_tile=lambda: tile, desc=types.SimpleNamespace(nz=64), step=lambda n: None,
                                set_tile=lambda **kw: timed.append(kw))
    tuning.autotune(sim, steps=1, reps=1)
    assert vars(tile) in timed
