"""The raster tile's entry in the tuner's cache names the shape and the tile kernel's blocks per
CU: one that names another occupancy was timed on another kernel, so it is timed again and
replaced; one that names a variant of this build is applied without timing."""
import pytest

from gpu_util import device_depos, make_plan, say
from paper_2104_08265_amd import synth

pytestmark = pytest.mark.gpu


def test_choice_of_another_kernel_is_timed_again(wct, tmp_path):
    wl = synth.config2(n_depos=500, n_tracks=3, n_ticks=480, wires=(48, 48, 70), fluctuate=True)
    dd, o = device_depos(wct, wl), wct.opts(3.0, True, 1, wl.seed)
    cache = tmp_path / "tune.txt"
    key = "wct-tile f32 3" + "".join(f" {p.n_wires} {p.n_ticks} {p.n_impacts}" for p in wl.planes) + " fluct 1 -> "
    names = {f"{v['th']} {v['tw']} {v['blocks_per_cu']}": v["index"] for v in wct.tile_variants() if v["dtype"] == "f32"}
    # the drawn tile kernel keeps a tile in 160 KB of LDS at most four times
    assert all(int(n.split()[2]) <= 4 for n in names)
    say("tile choices of another kernel")
    for name in ("128 48 5", "128 32 6"):
        assert name not in names
        cache.write_text(key + name + "\n")
        plan = make_plan(wct, wl)
        v = plan.tune_raster(dd, o, cache)
        lines = cache.read_text().splitlines()
        assert len(lines) == 2 and lines[1].startswith(key) and names[lines[1][len(key):]] == v
        plan.close()
    for name, index in names.items():
        cache.write_text(key + name + "\n")
        plan = make_plan(wct, wl)
        assert plan.tune_raster(dd, o, cache) == index and cache.read_text() == key + name + "\n"
        plan.close()
