"""The drawn-count tile kernel (Sec. 4.3.1) on windows of 1 and 4.2 sigma, bit for bit against the
oracle: the weights of its estimates and of the defining counts differ most at the edges of
wide windows, and times the electron count (up to 2^31) decides what an estimate may claim.
And widths next to the rounding of the position, whose edges round to five sigma, where the
defining series gives weights below 0 and above 1, on rows of one and two electrons."""
import numpy as np
import pytest

from gpu_util import device_depos, make_plan, say, to_np
from oracle import fluct as OF
from oracle import normal as ON
from paper_2104_08265_amd import synth
from test_gpu_raster_draw import workload

pytestmark = pytest.mark.gpu


def check(wct, where, n, dtype, mode, nsigma, wl=None):
    wl = wl or workload(where, n, dtype)
    plan = make_plan(wct, wl)
    ref = (OF.raster_fluct if mode == 1 else ON.raster_normal)(wl.depos, wl.planes, wl.seed, nsigma)[0][0]
    say("drawn tiles", dtype, where, n, "mode", mode, "nsigma", nsigma)
    got = to_np(plan.grid_view(plan.raster(device_depos(wct, wl), wct.opts(nsigma, mode, 1, wl.seed)))[0])
    if where == "huge" and dtype == "f32":  # FP32 cells round each addition past 2^24
        assert np.all(np.abs(got - ref) <= n * 2.0**-24 * ref)
    else:
        assert np.array_equal(got, ref)
    plan.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("where,n", [("any", 90), ("crowded", 300), ("huge", 40)])
@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("nsigma", [1.0, 4.2])
def test_drawn_tiles_of_narrow_and_wide_windows(wct, nsigma, mode, where, n, dtype):
    check(wct, where, n, dtype, mode, nsigma)


def off_range_workload(dtype):
    """Rows inside a cell whose edges lie x sqrt 2 sigma out, one unit in the last place of the
    position: erf(x) of the series is 0.6 to -6 there.  One axis or both."""
    xt, xp = np.meshgrid(np.linspace(4.92, 5.03, 30), [2.5] * 4 + list(np.linspace(4.95, 5.03, 9)))
    n = xt.size
    cell = 64 + np.arange(n) % 60, 64 + np.arange(n) // 60
    ulp = 2.0**-46  # of 64 to 128
    t, p = cell[0] + 0.5, (cell[1] + 0.5) / 10
    st, sp = ulp / (xt.ravel() * np.sqrt(2.0)), ulp / (xp.ravel() * np.sqrt(2.0)) / 10
    d = synth.Depos(1.0 + np.arange(n) % 2, t, p, st, np.where(xp.ravel() < 4, 1e-3, sp), np.zeros(n, np.int32),
                    np.zeros(n, np.int32), np.arange(n, dtype=np.int32))
    wl = workload("any", 1, dtype)
    return synth.Workload("off range", wl.planes, wl.responses, synth._finish(d, dtype), dtype=dtype, seed=3)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("mode", [1, 2])
def test_drawn_tiles_of_weights_outside_0_and_1(wct, mode, dtype):
    check(wct, "off range", 390, dtype, mode, 4.2, off_range_workload(dtype))
