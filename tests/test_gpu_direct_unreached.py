"""The direct wire pass where a block of eight wires per lane holds a tile that some row reaches
beside one that none reaches, with noise (pass C then reads every wire's spectrum) and without:
what the row pass left in the spectra of unreached rows must not show.  With 10 impacts per
pitch the row flags hide those rows, with 12 the tile flags alone do.  The workspace holds NaN
before the call.  Every event of a large call against the same event alone, whose smaller launch
takes four wires per lane and one tile per block, bit for bit; and against the oracle's signal
and noise at 1e-5 relative L2, the FP32 parity bar."""
import numpy as np
import pytest
import torch

from gpu_util import device_depos, make_plan, rel_l2, say, to_np
from oracle import convolve as OC
from oracle import noise as ON
from oracle import raster as OR
from paper_2104_08265_amd import synth

pytestmark = pytest.mark.gpu
EVENTS = 5  # 157 frequency chunks x 3 blocks x 5 events: past eight blocks per CU
TOL = 1e-5


def workload(wires, impacts, centres):
    """Per event (a list of wires) narrow depositions around its wires; L_t = 1250."""
    pl = synth.Plane(wires, 1024, impacts, 10, 200)
    rng = np.random.default_rng(wires + impacts)
    ev = np.concatenate([np.full(len(c), e) for e, c in enumerate(centres)]).astype(np.int32)
    p = np.concatenate([np.asarray(c, float) for c in centres])
    n = len(p)
    d = synth.Depos(rng.lognormal(8, 0.3, n), rng.uniform(100, 900, n), p, rng.uniform(0.5, 2, n),
                    rng.uniform(0.2, 0.5, n), np.zeros(n, np.int32), ev, np.arange(n, dtype=np.int32))
    return synth.Workload("unreached", [pl], [synth.make_response(pl, rng)], synth._finish(d, "f32"), dtype="f32")


def set_noise(plan, lt):
    amp = synth.noise_amplitude(lt, 50.0)
    plan.set_noise(0, amp)
    return amp


def nan_workspace(wct, plan, n_events, n_rows):
    plan.workspace(wct.OP_SIMULATE, n_events, n_rows)[0].fill_(0xFF)


@pytest.mark.parametrize("noise", [True, False])
@pytest.mark.parametrize("impacts", [10, 12])
@pytest.mark.parametrize("wires", [1030, 1280])
def test_mixed_blocks_write_exact_zeros(wct, wires, impacts, noise):
    # one, two, three and five reached tiles of five, and an event without charge
    centres = [[130.0], [60.0, 800.0], [253.0, 900.0], [100.5, 300.5, 600.5, 900.5, 1027.0], []]
    wl = workload(wires, impacts, centres)
    many, one = make_plan(wct, wl, max_events=EVENTS), make_plan(wct, wl)
    lt = many.plane_info(0)["lt"]
    amp = set_noise(many, lt)
    set_noise(one, lt)
    dd = device_depos(wct, wl)
    nan_workspace(wct, many, EVENTS, dd.n)
    say("unreached tiles", wires, impacts, "noise", noise)
    got = many.simulate(dd, wct.opts(3.0, False, EVENTS, 9, noise=noise)).view(EVENTS, -1)
    R = synth.round_responses(wl)[0].astype(np.float64)
    grids = OR.raster(wl.depos, wl.planes, n_events=EVENTS)
    for e in range(EVENTS):
        nan_workspace(wct, one, 1, dd.n)
        ref = one.simulate(dd, wct.opts(3.0, False, 1, 9, event_base=e, noise=noise))
        assert torch.equal(got[e], ref), e
        if e not in (0, 2):
            continue
        M = OC.convolve_fft(grids[e][0], R, impacts)
        if noise:
            M = M + ON.noise_waveforms(amp, 9, e, 0, wires, 1024, lt)
        assert rel_l2(to_np(got[e]).reshape(M.shape), M) < TOL, e
    many.close()
    one.close()

