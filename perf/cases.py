"""Performance cases of the signal simulation, through the package's public entry points.

Each case is one pass of a program that holds a plan (geometry and wire responses) and
device buffers and calls wct.Plan / torch_ops as the benchmark and the tests do:

* simulate - rasterise depositions and convolve with the wire response (one or more events);
* graph    - the same replayed through the plan's own graph cache;
* chain    - 3D depositions drifted onto the planes, then simulated with noise;
* raster   - the charge grid alone;
* convolve - a given grid to waveforms;
* fit      - forward and backward of the differentiable simulation;
* digitize - ADC codes of given waveforms.

Geometries: "plane" (one plane, points or straight tracks in the (pitch, tick) plane),
"box" (MicroBooNE-like, three planes) and "faces" (two DUNE-like faces of three planes).
"""
import math

import numpy as np
import torch

from paper_2104_08265_amd import synth, torch_ops, wct

DEVICE = "cuda:0"
NSIGMA = 3.0


def _case(name, op, geometry, wires, ticks, depos, pattern, mode=0, dtype="f32", events=1, noise=False,
          half_wires=10, impacts=10, resp_ticks=200):
    c = {"op": op, "geometry": geometry, "wires": wires, "ticks": ticks, "depos": depos, "pattern": pattern,
         "mode": mode, "dtype": dtype, "events": events, "noise": noise, "half_wires": half_wires,
         "impacts": impacts, "resp_ticks": resp_ticks}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a thousand points on one FP64 plane, where launches count
        _case("point_cloud_f64", "simulate", "plane", "256", 1024, 1000, "points", dtype="f64"),
        # a small triggered event replayed from the plan's graph, as a serving loop does
        _case("graph_small_event", "graph", "box", "600,600,864", 2400, 2000, "tracks", mode=1),
        # one step of a fit of deposition parameters on one plane
        _case("fit_small", "fit", "plane", "256", 1024, 20000, "tracks"),
        # one step of a fit on a three-plane detector of middle size
        _case("fit_tracks", "fit", "box", "800,800,1152", 6000, 50000, "tracks"),
        # a geometry nobody tuned: odd sizes, a response of 15 wires, FP64
        _case("ragged_f64", "simulate", "plane", "479", 2999, 5000, "points", dtype="f64", half_wires=7,
              resp_ticks=151),
        # the mean charge grid of a cosmic-ray event (the rasterisation step alone)
        _case("raster_mean_tracks", "raster", "box", "2400,2400,3456", 9600, 100000, "tracks"),
        # the full event of the benchmark: three planes, 1e5 depositions, binomial counts
        _case("simulate_tracks", "simulate", "box", "2400,2400,3456", 9600, 100000, "tracks", mode=1),
        # the largest: crowded electromagnetic showers on two faces, 1e6 depositions
        _case("simulate_showers", "simulate", "faces", "800,800,960", 6000, 1000000, "showers", mode=1),
        # 3D depositions through drift, normal-approximation counts, noise
        _case("chain_normal_noise", "chain", "box", "2400,2400,3456", 9600, 100000, "tracks", mode=2, noise=True),
        # a batch of sparse and crowded events in one call
        _case("batch_events", "simulate", "box", "2400,2400,3456", 9600, 200000, "mixed", mode=1, events=16),
        # waveforms of grids made elsewhere (charge everywhere), six planes
        _case("convolve_dense", "convolve", "faces", "800,800,960", 6000, 0, "dense"),
        # ADC codes of an event's waveforms
        _case("digitize_event", "digitize", "box", "2400,2400,3456", 9600, 0, "dense"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["simulate", "simulate", "simulate", "simulate", "raster", "raster", "fit", "fit", "graph",
                     "chain", "convolve", "digitize"])
    geometry = rng.choice(["plane", "box", "faces"])
    if op == "chain":
        geometry = "box"
    dtype = rng.choice(["f32", "f32", "f32", "f64"])
    if op in ("graph", "chain"):
        dtype = "f32"
    if geometry == "plane":
        wires, ticks = str(_log_int(rng, 48, 1500)), _log_int(rng, 300, 6000)
    elif geometry == "box":
        w = _log_int(rng, 96, 2400 if dtype == "f32" else 800)
        wires, ticks = "%d,%d,%d" % (w, w, int(1.44 * w)), _log_int(rng, 600, 9600 if dtype == "f32" else 4800)
    else:
        w = _log_int(rng, 96, 800)
        wires, ticks = "%d,%d,%d" % (w, w, int(1.2 * w)), _log_int(rng, 600, 6000 if dtype == "f32" else 3000)
    mode = rng.choice([0, 1, 1, 2]) if dtype == "f32" else rng.choice([0, 0, 1])
    pattern = rng.choice(["tracks", "showers"]) if geometry != "plane" else rng.choice(["points", "tracks"])
    events = rng.choice([1, 1, 1, 2, 5, 16]) if op == "simulate" and geometry == "box" else 1
    depos = _log_int(rng, 100, 200000 if geometry != "plane" else 20000)
    half_wires = rng.choice([10, 10, 10, 5])
    noise = op == "chain" or (op == "simulate" and rng.random() < 0.25)
    if op == "fit":
        mode, noise = 0, False
        depos = min(depos, 50000)
    if op in ("convolve", "digitize"):
        mode, pattern, depos = 0, "dense", 0
    if events > 1:
        pattern = "mixed"
    return _case(None, op, geometry, wires, ticks, depos, pattern, mode, dtype, events, noise, half_wires,
                 resp_ticks=rng.choice([200, 200, 120, 151]))


# -- inputs -----------------------------------------------------------------------------

def _wires(case):
    return tuple(int(w) for w in case["wires"].split(","))


def _geometry(case):
    """(detector or None, planes) of a case."""
    w = _wires(case)
    if case["geometry"] == "plane":
        det, planes = None, [synth.Plane(w[0], case["ticks"], kind="collection")]
    elif case["geometry"] == "box":
        det = synth.detector_uboone_like(case["ticks"], w)
        planes = det.planes
    else:
        det = synth.detector_dune_like(case["ticks"], w)
        planes = list(det.planes) + [synth.Plane(p.n_wires, p.n_ticks, kind=p.kind) for p in det.planes]
    for p in planes:
        p.n_impacts, p.half_wires, p.resp_ticks = case["impacts"], case["half_wires"], case["resp_ticks"]
    return det, planes


def _points3d(rng, det, pattern, n):
    """Positions (cm), times (ticks), charges and a group number of n 3D depositions."""
    if pattern == "tracks":
        n_tracks = max(1, math.ceil(n / 2000))
        xyz, t0 = synth.track_points(rng, det, n_tracks, n)
        return xyz, t0, synth.moyal_charge(rng, n, 6000.0), np.arange(n) * n_tracks // max(n, 1)
    margin = min(80.0, 0.1 * min(p.n_wires for p in det.planes))
    xyz, t0, sid = synth.shower_points(rng, det, max(1, math.ceil(n / 50000)), n, margin=margin)
    return xyz, t0, synth.lognormal_charge(rng, n, 3000.0), sid


def _event(rng, case, det, planes, pattern, n, event):
    """Depo-plane rows of one event."""
    ids = np.arange(n)
    if det is None:
        if pattern == "points":
            return synth.uniform_points(rng, 0, planes[0], n, event=event)
        size = [planes[0].n_wires, planes[0].n_ticks]
        a, b = rng.uniform([0, 0], size, (20, 2)), rng.uniform([0, 0], size, (20, 2))
        at = a[ids % 20] + rng.uniform(0.0, 1.0, n)[:, None] * (b - a)[ids % 20]
        return synth.Depos(synth.lognormal_charge(rng, n, 5000.0), at[:, 1], at[:, 0], rng.uniform(1.0, 3.0, n),
                           rng.uniform(0.3, 2.0, n), np.zeros(n, np.int32), np.full(n, event, np.int32),
                           ids.astype(np.int32))
    xyz, t0, q, group = _points3d(rng, det, pattern, n)
    faces = 2 if case["geometry"] == "faces" else 1
    parts = []
    for f in range(faces):
        m = group % faces == f
        if m.any():
            parts.append(synth._rows_from_points(det, xyz[m], t0[m], q[m], event, ids[m], plane_offset=3 * f))
    return synth.Depos.concat(parts)


def _float(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _inputs(case, seed):
    """What the case's program is given: numpy depositions or 3D points, and host responses."""
    rng = np.random.default_rng(seed)
    det, planes = _geometry(case)
    npdt = np.float32 if case["dtype"] == "f32" else np.float64
    responses = [synth.make_response(p, rng).astype(npdt) for p in planes]
    depos = points = None
    if case["op"] == "chain":
        xyz, t0, q, _ = _points3d(rng, det, case["pattern"], case["depos"])
        n = case["depos"]
        points = synth.Points(xyz[:, 0], xyz[:, 1], xyz[:, 2], 0.5 * t0, q, rng.uniform(0.03, 0.06, n),
                              rng.uniform(0.03, 0.06, n), np.zeros(n, np.int32), np.arange(n, dtype=np.int32))
        points = points.astype(npdt)
    elif case["op"] not in ("convolve", "digitize"):
        parts = []
        for e in range(case["events"]):
            pattern, n = case["pattern"], case["depos"]
            if pattern == "mixed":  # log-uniform counts, tracks and showers
                n = int(round(math.exp(rng.uniform(math.log(100), math.log(max(n, 101))))))
                pattern = "tracks" if rng.uniform() < 0.5 else "showers"
            parts.append(_event(rng, case, det, planes, pattern, n, e))
        depos = synth.Depos.concat(parts).astype(npdt)
    return det, planes, responses, depos, points


def _dense(case, seed, n):
    """Charge everywhere (convolve) or waveform samples (digitize), made on the GPU."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    if case["op"] == "convolve":
        return torch.empty(n, dtype=_float(case), device=DEVICE).exponential_(0.01, generator=g)
    return torch.empty(n, dtype=_float(case), device=DEVICE).normal_(0.0, 3.0e4, generator=g)


def prepare(case, seed):
    det, planes, responses, depos, points = _inputs(case, seed)
    plan = wct.Plan(planes, responses, dtype=case["dtype"], max_events=min(case["events"], 8))
    s = {"case": case, "plan": plan,
         "opts": wct.opts(NSIGMA, case["mode"], case["events"], seed=seed, noise=case["noise"])}
    if case["noise"]:
        for k, info in enumerate(plan.info):
            plan.set_noise(k, synth.noise_amplitude(info["lt"], 300.0))
    if depos is not None:
        s["depos"] = wct.DeviceDepos.from_numpy(depos, DEVICE, plan.torch_dtype)
    if points is not None:
        s["points"] = wct.DevicePoints.from_numpy(points, DEVICE, plan.torch_dtype)
        s["drift"] = wct.drift_params(*synth.drift_params(det).values())
    if case["op"] == "graph":
        s["wave"] = plan.new_wave(case["events"])
    elif case["op"] == "convolve":
        s["grid"] = _dense(case, seed, plan.grid_elems)
    elif case["op"] == "digitize":
        s["wave"] = _dense(case, seed, plan.wave_elems)
        for k, p in enumerate(planes):
            plan.set_adc(k, 1.0 / 40.0, 900.0 if p.kind == "collection" else 2048.0, 4095)
    elif case["op"] == "fit":
        d = s["depos"]
        s["target"] = plan.new_wave().normal_(0.0, 100.0, generator=torch.Generator(device=DEVICE).manual_seed(seed))
        s["leaves"] = [x.requires_grad_() for x in (d.q, d.t, d.p, d.sigma_t, d.sigma_p)]
    return s


def run(state):
    case, plan = state["case"], state["plan"]
    op = case["op"]
    if op == "simulate":
        return plan.simulate(state["depos"], state["opts"])
    if op == "graph":
        return plan.simulate_graph(state["depos"], state["opts"], state["wave"])
    if op == "chain":
        return plan.simulate(plan.drift(state["points"], state["drift"]), state["opts"])
    if op == "raster":
        return plan.raster(state["depos"], state["opts"])
    if op == "convolve":
        return plan.convolve(state["grid"])
    if op == "digitize":
        return plan.digitize(state["wave"])
    d = state["depos"]
    wave = torch_ops.simulate(plan, *state["leaves"], d.plane, d.event, d.depo_id, NSIGMA)
    loss = 0.5 * (wave - state["target"]).square().sum()
    return [wave.detach(), *torch.autograd.grad(loss, state["leaves"])]


# -- what a pass cannot do without --------------------------------------------------------

def _cells_per_row(case):
    """Mean cells of a row's 3-sigma window for the widths the inputs are drawn with."""
    if case["geometry"] == "plane":
        return (6 * 2.0 + 1) * (6 * case["impacts"] * 1.15 + 1)
    if case["op"] == "chain":
        return 600.0
    s = [math.sqrt((k + 0.5) / 100) for k in range(100)]
    return sum((6 * (1 + 2 * x) + 1) * (6 * case["impacts"] * (0.3 + 1.7 * x) + 1) for x in s) / len(s)


def work(case):
    _, planes = _geometry(case)
    size = 4 if case["dtype"] == "f32" else 8
    events = case["events"]
    grid = sum(p.n_wires * p.n_impacts * p.n_ticks for p in planes) * size * events
    wave = sum(p.n_wires * p.n_ticks for p in planes) * size * events
    if case["pattern"] == "mixed":
        top = max(case["depos"], 101)
        per_event = (top - 100) / math.log(top / 100)
    else:
        per_event = case["depos"]
    rows = per_event * events * (len(planes) / (2 if case["geometry"] == "faces" else 1))
    row_bytes = rows * (5 * size + 12)
    cells = rows * _cells_per_row(case)
    raster = cells * {0: 3, 1: 60, 2: 90}[case["mode"]]  # mean product and add; generator, probability, draw
    conv = 0.0
    for p in planes:
        lt = p.n_ticks + p.resp_ticks - 1
        lw = p.n_wires + p.half_wires
        conv += (p.n_impacts + 1) * p.n_wires * 2.5 * lt * math.log2(lt)
        conv += (lt / 2 + 1) * lw * ((p.n_impacts + 1) * 5 * math.log2(lw) + 8 * p.n_impacts)
    conv *= events
    op = case["op"]
    if op == "raster":
        return {"bytes": row_bytes + grid, "flops": raster}
    if op == "convolve":
        return {"bytes": grid + wave, "flops": conv}
    if op == "digitize":
        return {"bytes": wave + wave / size * 2, "flops": 3 * wave / size}
    if op == "fit":
        return {"bytes": 2 * row_bytes + 5 * rows * size + 3 * wave, "flops": 2 * conv + raster + 12 * cells}
    if op == "chain":
        return {"bytes": case["depos"] * (7 * size + 8) + wave, "flops": raster + conv}
    return {"bytes": row_bytes + wave, "flops": raster + conv}


# -- the same in 64 bits, by plain torch --------------------------------------------------

def _edges(mu, sigma, b0, n, size):
    """Gaussian integrals over the bins b0 .. b0 + n - 1 inside [mu - 3 sigma, mu + 3 sigma] and the axis."""
    lo, hi = mu - NSIGMA * sigma, mu + NSIGMA * sigma
    first, last = torch.floor(lo.detach()).clamp(min=0), torch.ceil(hi.detach()).clamp(max=size)
    x = b0[:, None] + torch.arange(n + 1, device=mu.device, dtype=mu.dtype)
    x = torch.minimum(x, last[:, None])
    x = torch.minimum(torch.maximum(x, lo[:, None]), hi[:, None])
    e = torch.erf((x - mu[:, None]) / (math.sqrt(2.0) * sigma[:, None]))
    w = 0.5 * (e[:, 1:] - e[:, :-1])
    inside = (b0[:, None] + torch.arange(n, device=mu.device) < last[:, None]) & (last > first)[:, None]
    return torch.where(inside, w, torch.zeros_like(w))


def _exact_patches(plane, t, p, st, sp):
    """(A [n, nb], B [n, nk], first row, first tick) of rows of one plane."""
    I, nb, nt = plane.n_impacts, plane.n_impacts * plane.n_wires, plane.n_ticks
    u, su = I * p, I * sp
    b0 = torch.floor((u - NSIGMA * su).detach()).clamp(min=0)
    k0 = torch.floor((t - NSIGMA * st).detach()).clamp(min=0)
    wide = int((torch.ceil((u + NSIGMA * su).detach()) - b0).max().clamp(min=1))
    long = int((torch.ceil((t + NSIGMA * st).detach()) - k0).max().clamp(min=1))
    return _edges(u, su, b0, wide, nb), _edges(t, st, k0, long, nt), b0.long(), k0.long()


def _exact_cells(plane, b0, k0, nb, nk):
    """Flat grid indices of a patch's cells (cells off the grid, whose weight is 0, on cell 0)."""
    b = b0[:, None] + torch.arange(nb, device=b0.device)
    k = k0[:, None] + torch.arange(nk, device=b0.device)
    at = b[:, :, None] * plane.n_ticks + k[:, None, :]
    off = (b >= plane.n_impacts * plane.n_wires)[:, :, None] | (k >= plane.n_ticks)[:, None, :]
    return torch.where(off, torch.zeros_like(at), at)


CHUNK = 8192


def _exact_grid(plane, rows):
    q, t, p, st, sp = rows
    grid = torch.zeros(plane.n_impacts * plane.n_wires * plane.n_ticks, dtype=torch.float64, device=DEVICE)
    for a in range(0, q.numel(), CHUNK):
        c = slice(a, a + CHUNK)
        A, B, b0, k0 = _exact_patches(plane, t[c], p[c], st[c], sp[c])
        v = (q[c, None] * A)[:, :, None] * B[:, None, :]
        grid.index_add_(0, _exact_cells(plane, b0, k0, A.shape[1], B.shape[1]).reshape(-1), v.reshape(-1))
    return grid


def _smooth(n):
    while True:
        m = n
        for f in (2, 3, 5):
            while m % f == 0:
                m //= f
        if m == 1:
            return n
        n += 1


def _spectra(plane, response):
    """Per impact phase the 2D spectrum of the response, wire offset k at index -k."""
    K, lw, lt = plane.half_wires, _smooth(plane.n_wires + plane.half_wires), _smooth(plane.n_ticks + plane.resp_ticks)
    r = torch.as_tensor(response, device=DEVICE).double()
    for i in range(plane.n_impacts):
        h = torch.zeros(lw, lt, dtype=torch.float64, device=DEVICE)
        h[(-torch.arange(-K, K + 1, device=DEVICE)) % lw, : plane.resp_ticks] = r[:, i]
        yield torch.fft.fft(torch.fft.rfft(h, dim=1), dim=0)


def _exact_convolve(plane, response, grid):
    I, nw, nt = plane.n_impacts, plane.n_wires, plane.n_ticks
    lw, lt = _smooth(nw + plane.half_wires), _smooth(nt + plane.resp_ticks)
    g = grid.view(nw, I, nt)
    total = None
    for i, spec in enumerate(_spectra(plane, response)):
        s = torch.fft.fft(torch.fft.rfft(g[:, i], n=lt, dim=1), n=lw, dim=0) * spec
        total = s if total is None else total.add_(s)
    return torch.fft.irfft(torch.fft.ifft(total, dim=0)[:nw], n=lt, dim=1)[:, :nt].reshape(-1)


def _exact_adjoint(plane, response, gwave):
    I, nw, nt = plane.n_impacts, plane.n_wires, plane.n_ticks
    lw, lt = _smooth(nw + plane.half_wires), _smooth(nt + plane.resp_ticks)
    s = torch.fft.fft(torch.fft.rfft(gwave.view(nw, nt), n=lt, dim=1), n=lw, dim=0)
    out = torch.empty(nw, I, nt, dtype=torch.float64, device=DEVICE)
    for i, spec in enumerate(_spectra(plane, response)):
        out[:, i] = torch.fft.irfft(torch.fft.ifft(s * spec.conj(), dim=0)[:nw], n=lt, dim=1)[:, :nt]
    return out.reshape(-1)


def _exact_gradients(plane, rows, H):
    got = [[] for _ in rows]
    for a in range(0, rows[0].numel(), CHUNK):
        q, t, p, st, sp = leaves = [x[a:a + CHUNK].clone().requires_grad_() for x in rows]
        A, B, b0, k0 = _exact_patches(plane, t, p, st, sp)
        h = H[_exact_cells(plane, b0, k0, A.shape[1], B.shape[1])]
        loss = (q[:, None] * A * (h * B[:, None, :]).sum(2)).sum()
        for g, x in zip(got, torch.autograd.grad(loss, leaves)):
            g.append(x)
    return [torch.cat(g) for g in got]


def exact(case, seed):
    if case["mode"] != 0 or case["noise"] or case["op"] in ("digitize", "chain"):
        return None  # drawn counts, drawn noise and ADC codes are compared as they are
    _, planes, responses, depos, _ = _inputs(case, seed)
    if case["op"] == "convolve":
        grid = _dense(case, seed, sum(p.n_impacts * p.n_wires * p.n_ticks for p in planes))
        sizes = [p.n_impacts * p.n_wires * p.n_ticks for p in planes]
        return torch.cat([_exact_convolve(p, r, g.double()) for p, r, g in zip(planes, responses, grid.split(sizes))])
    f = [torch.as_tensor(x, device=DEVICE).double() for x in (depos.q, depos.t, depos.p, depos.sigma_t, depos.sigma_p)]
    where = [torch.as_tensor(x, device=DEVICE) for x in (depos.event, depos.plane)]
    at = [[(where[0] == e) & (where[1] == k) for k in range(len(planes))] for e in range(case["events"])]
    grids = [[_exact_grid(p, [x[m] for x in f]) for p, m in zip(planes, ms)] for ms in at]
    if case["op"] == "raster":
        return torch.cat([g for gs in grids for g in gs])
    wave = torch.cat([_exact_convolve(p, r, g) for gs in grids for p, r, g in zip(planes, responses, gs)])
    if case["op"] != "fit":
        return wave
    del grids
    target = torch.empty(wave.numel(), dtype=_float(case), device=DEVICE)
    target.normal_(0.0, 100.0, generator=torch.Generator(device=DEVICE).manual_seed(seed))
    back = (wave - target.double()).split([p.n_wires * p.n_ticks for p in planes])
    grads = [torch.zeros_like(x) for x in f]
    for p, r, g, m in zip(planes, responses, back, at[0]):
        if m.any():
            for to, x in zip(grads, _exact_gradients(p, [x[m] for x in f], _exact_adjoint(p, r, g))):
                to[m] = x
    return [wave, *grads]
