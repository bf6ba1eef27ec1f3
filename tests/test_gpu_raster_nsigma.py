"""The drawn-count tile kernel (Sec. 4.3.1) on windows of 1 and 4.2 sigma, bit for bit against the
oracle: the weights of its estimates and of the defining counts differ most at the edges of
wide windows, and times the electron count (up to 2^31) decides what an estimate may claim."""
import numpy as np
import pytest

from gpu_util import device_depos, make_plan, say, to_np
from oracle import fluct as OF
from oracle import normal as ON
from test_gpu_raster_draw import workload

pytestmark = pytest.mark.gpu


def check(wct, where, n, dtype, mode, nsigma):
    wl = workload(where, n, dtype)
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
