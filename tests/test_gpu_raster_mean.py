"""The mean raster's matrix-core tile kernel (Sec. 2.1.1) against the FP64 oracle where it
can go wrong: windows at every offset from the 16 x 16 blocks and the tiles, tiles cut by
the grid's edges (odd sizes), row counts around the 16 staged at a time and past one work
item (split tiles), windows beyond 4.2 sigma (the library's erf instead of the polynomial),
and every tile shape.

Tolerances (relative L2 of a plane): FP64 weights are differences of erf values near 1, each
within a few 1e-16 on both sides, of weights of 1e-2 and more: 1e-12.  FP32 grids round each
cell once, or once more per work item of a split tile (at most three here): 3e-7.
"""
import numpy as np
import pytest

from gpu_util import device_depos, make_plan, rel_l2, say, to_np
from oracle import raster as OR
from paper_2104_08265_amd import synth

pytestmark = pytest.mark.gpu

TOL = {"f32": 3e-7, "f64": 1e-12}


def workload(dtype, n, wires, ticks, where):
    rng = np.random.default_rng(n + wires)
    pl = synth.Plane(wires, ticks, 10, 2, 12)
    if where == "crowded":  # every row around one tile corner
        p, t = rng.uniform(12.5, 13.1, n), rng.uniform(47.0, 49.0, n)
    else:
        p, t = rng.uniform(-0.5, wires + 0.5, n), rng.uniform(-3.0, ticks + 3.0, n)
    d = synth.Depos(rng.lognormal(7, 0.5, n), t, p, rng.uniform(0.4, 3.0, n), rng.uniform(0.05, 1.2, n),
                    np.zeros(n, np.int32), np.zeros(n, np.int32), np.arange(n, dtype=np.int32))
    return synth.Workload("mean", [pl], [synth.make_response(pl, rng)], synth._finish(d, dtype), dtype=dtype)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n,wires,ticks,where", [(1, 13, 97, "all"), (17, 26, 145, "all"), (900, 39, 193, "all"),
                                                 (15, 26, 100, "crowded"), (600, 26, 100, "crowded")])
@pytest.mark.parametrize("nsigma", [3.0, 4.2, 6.0])
def test_mean_tiles_equal_the_oracle(wct, dtype, n, wires, ticks, where, nsigma):
    wl = workload(dtype, n, wires, ticks, where)
    plan = make_plan(wct, wl)
    dd = device_depos(wct, wl)
    ref = OR.raster(wl.depos, wl.planes, nsigma)[0][0]
    for v in plan.tile_candidates():
        plan.set_tile(v)
        say("mean tiles", dtype, n, wires, ticks, where, nsigma, "tile", v)
        got = to_np(plan.grid_view(plan.raster(dd, wct.opts(nsigma, False)))[0])
        assert rel_l2(got, ref) < TOL[dtype], v
    plan.close()
