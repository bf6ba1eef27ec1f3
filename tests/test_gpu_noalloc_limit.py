"""wct_raster_noalloc next to the size of its static scratch, with few rows over many tiles: the
raster's workspace has the size it has had from the first layout on (64 control words and the
tiles' counts, two lists of four slots a row, two offsets and an item a tile, an item per 256
rows, a word a row, the scans' sums; each rounded to 256 bytes), so the calls that fit are the
same ones.  The last call that fits gives wct_raster's grid, the next one is refused."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_2104_08265_amd import synth

pytestmark = pytest.mark.gpu
PLANES, TICKS = 8, 9600  # one impact row each: a tile of 128 x 48 holds 48 cells


def size(tiles, rows):
    words = lambda n: -(-4 * n // 256) * 256
    return (words(64 + tiles) + 2 * words(4 * rows) + 2 * words(tiles + 1) + words(tiles + -(-4 * rows // 256) + 1) +
            words(rows) + words(2 * max(-(-tiles // 4096), 1)))


def test_noalloc_raster_at_the_scratch_limit(wct):
    pl = synth.Plane(1, TICKS, 1, 1, 16)
    limit = wct.NOALLOC_SCRATCH_BYTES
    tiles_ev = PLANES * (TICKS // 48)
    events = next(e for e in range(1, 10**5) if size((e + 1) * tiles_ev, 1) > limit)
    plan = wct.Plan([pl] * PLANES, [np.ones((3, 1, 16))] * PLANES, dtype="f32", max_events=events)
    v = next(v for v in wct.tile_variants() if (v["dtype"], v["th"], v["tw"]) == ("f32", 128, 48))
    plan.set_tile(v["index"])
    last = next(n for n in range(1, 2000) if size(events * tiles_ev, n + 1) > limit)
    for n in (1, 100, last - 1, last, last + 1):
        assert wct.wct_workspace_bytes(plan.h, wct.OP_RASTER, events, n) == size(events * tiles_ev, n), n
    rng = np.random.default_rng(last)
    n = last + 1
    d = synth.Depos(np.full(n, 1000.0), rng.uniform(0, TICKS, n), rng.uniform(0, 1, n), rng.uniform(0.5, 20, n),
                    rng.uniform(0.2, 0.6, n), rng.integers(0, PLANES, n).astype(np.int32),
                    rng.integers(0, events, n).astype(np.int32), np.arange(n, dtype=np.int32))
    dd = wct.DeviceDepos.from_numpy(synth._finish(d, "f32"), "cuda:0", torch.float32)
    o = wct.opts(3.0, True, events, 5)
    say("noalloc raster at the limit:", events, "events", last, "rows")
    grid = plan.new_grid(events).fill_(-7.0)
    plan.raster_noalloc(dd.slice(0, last), o, grid)
    assert torch.equal(grid, plan.raster(dd.slice(0, last), o)) and torch.any(grid)
    with pytest.raises(wct.WctError) as e:
        plan.raster_noalloc(dd, o, grid)
    assert e.value.code == wct.WCT_E_WORKSPACE
    plan.close()
