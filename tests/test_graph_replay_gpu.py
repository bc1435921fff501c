"""Graph replay of whole record intervals on a one-pass tile that is the
caller's own choice (on the default one these grids step on bricks, which
replay nothing): several replays with other work between them, each checked
against plain launches of the same tile, whose calls are cut where the replay
begins and ends (the last of an odd number of steps is two half-steps, whose
sums are added in another order).  That the graph ran is read from the
device record counter, the last 256-byte slot of the workspace: only replays
write it."""
import pytest
import torch

from paper_2401_07416_amd import tdse

pytestmark = pytest.mark.gpu

N, H, STEPS = (64, 48, 56), 10, 150
TILES = [dict(fused=1, two_step=0, fused_rows=2, fused_zc=8, fused_threads=128, fused_prefetch=0),
         dict(fused=1, two_step=0, fused_rows=3, fused_zc=16, fused_threads=256, fused_prefetch=1)]


def make(prec, tile, stream, graph):
    d = tdse.make_desc(*N, 0.2, 0.21, 0.22, 0.6582119569, 0.0568563, precision=prec, k_det=N[2] // 2,
                       record_every=H, max_records=STEPS // H + 1, flags=tdse.FLAG_PIXEL_INTEGRAL)
    s = tdse.Sim(d, stream=stream)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    r = [torch.rand((N[2], N[1], N[0]), generator=g, device="cuda", dtype=torch.float64) for _ in range(3)]
    s.v.copy_(-30.0 * r[0])
    torch.cuda.synchronize()
    s.set_cap_quadratic(8, 8, 50.0)
    s.finalize()
    s.set_state(r[1] - 0.5, r[2] - 0.5, step=0)
    s.set_tile(graph=graph, **tile)
    return s


def counter(s):
    return int(s.workspace[-256:-248].view(torch.int64).item())


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("tile", TILES)
def test_every_replay_matches_plain_launches(prec, tile):
    print("graph replay", prec, tile, flush=True)
    plain = make(prec, tile, None, 0)
    side = torch.cuda.Stream()
    g = make(prec, tile, side, 1)
    done = 0
    # intervals replayed by each call, and what the counter then holds
    for n, replays in ((7, 0), (43, 4), (60, 6), (5, 0), (35, 3)):
        pre = min(-done % H, n)
        for k in (pre, (n - pre) // H * H, (n - pre) % H):
            plain.step(k)
        g.step(n)
        torch.cuda.synchronize()
        done += n
        if replays:
            assert counter(g) == done // H + 1
        for a, b in ((plain.psi_r, g.psi_r), (plain.psi_i, g.psi_i), (plain.records, g.records),
                     (plain.pixel, g.pixel), (plain.scalars, g.scalars)):
            assert torch.equal(a, b)
        assert plain.detect().flux == g.detect().flux
        # work of the caller's own between two replays
        torch.rand(1 << 20, device="cuda").sum().item()
    assert counter(plain) == 0 and g.detect().step == done == STEPS
