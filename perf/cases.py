"""The work that users of this library have it do, as measurable cases.

Three kinds, each through the public Python entry points:

* ``transport``  Monte Carlo runs of one chamber or of a batch (``Plan.run``, the one-call ``run`` and
  ``run_noalloc_into``), FP32 and FP64, from the 1e5-atom run of a single target to the 64-chamber sweep;
* ``fit``        one step of a power or rate fit: composition map and squared distance, forward and backward;
* ``inversion``  the chain after the runs of a tilt sweep: areas, compositions, d_e^2, covered area, fits.

``listed`` gives the fixed cases, ``draw`` others of the same ranges, ``prepare`` what a program holds before
the call, ``run`` one pass, ``work`` the bytes and operations it cannot do without, ``exact`` the 64-bit values
of the outputs that have some (a Monte Carlo tally has none: its whole numbers stay what they are).
"""
import math

import numpy as np
import torch

import paper_2411_14413_amd as spx
import sputter_inputs as si

# Mean history of an atom from the FP64 oracle, by pressure [Pa]: collisions, diffusive steps, thermalised
# share, for the single target and for four confocal cathodes (25 deg, 150 mm).
HISTORY_P = (0.1, 0.25, 0.5, 1.0, 2.0)
HISTORY = {
    "single": ((1.597, 4.202, 8.170, 12.05, 13.86), (0.3, 6.3, 65.2, 467.0, 2273.0), (0.026, 0.145, 0.437, 0.767, 0.919)),
    "confocal": ((1.589, 4.255, 8.677, 14.90, 19.22), (0.1, 3.4, 45.9, 491.0, 3104.0), (0.012, 0.076, 0.266, 0.633, 0.901)),
    # chimneys around the targets and the other targets absorbing
    "chimneys": ((0.784, 2.063, 4.224, 7.541, 10.89), (0.0, 0.9, 11.4, 107.9, 578.0), (0.005, 0.031, 0.110, 0.272, 0.434)),
}
# Lane operations of a launch, a ballistic flight, a collision and a diffusive step (a 32-bit wide product or
# a transcendental counted as four).
OPS_LAUNCH, OPS_FLIGHT, OPS_COLLISION, OPS_STEP = 310, 292, 282, 90

SWEEP_SEED = 0
TILTS = (11.0, 14.5)


def transport(system, n, pressure=0.5, tilt=25.0, distance=150.0, grid=200, chambers=1, entry="run", precision=32,
              autotune=False, records=False, arrivals=False, chimneys=False, measured=False):
    return dict(kind="transport", system=system, n=int(n), pressure=float(pressure), tilt=float(tilt),
                distance=float(distance), grid=int(grid), chambers=int(chambers), entry=entry, precision=int(precision),
                autotune=autotune, records=records, arrivals=arrivals, chimneys=chimneys, measured=measured)


def fit(B, J, K):
    return dict(kind="fit", B=int(B), J=int(J), K=int(K))


def inversion(T, grid, areas, pitch, n):
    return dict(kind="inversion", T=int(T), grid=int(grid), areas=int(areas), pitch=float(pitch), n=int(n))


def listed():
    def named(name, case):
        return dict(case, name=name)
    return [
        # the smallest run in use: one target, 1e5 atoms, as an interactive look at a geometry
        named("single_1e5", transport("single", 1e5, grid=50)),
        # the benchmark's default: one target at 0.5, 0 and 2 Pa, 1e7 atoms each, a tuned plan replayed
        named("legs_3e7", transport("legs", 3e7, grid=50, autotune=True)),
        # a quaternary library: four confocal cathodes, atoms in proportion to the powers
        named("quaternary_2.3e7", transport("quaternary", 2.3e7)),
        # a design sweep: 64 four-cathode chambers in one launch, the largest run in use
        named("sweep_64", transport("sweep", 167342381, chambers=64)),
        # a detailed chamber: chimneys, cross absorption, a measured racetrack, every optional output
        named("chimneys_records", transport("quaternary", 2.3e6, chimneys=True, measured=True, records=True, arrivals=True)),
        # one run of a new geometry, its plan made for the call: a user's geometry scan
        named("new_geometry", transport("quaternary", 2.3e6, entry="once")),
        # the entry point that allocates nothing, as in a serving loop: several rounds of its fixed queue
        named("noalloc_4.6e6", transport("quaternary", 4.6e6, entry="noalloc")),
        # the FP64 reference run of one target, and of the three pressures
        named("fp64_single_1e5", transport("single", 1e5, grid=50, precision=64)),
        named("fp64_legs_9e5", transport("legs", 9e5, grid=50, precision=64)),
        # a step of a power fit at the 342 areas: a batch of 1024 power vectors
        named("fit_1024", fit(1024, 342, 4)),
        # the same over a screening batch
        named("fit_32768", fit(32768, 342, 4)),
        # the tilt inversion of a ternary library: 8 tilts, 342 areas of a 200 x 200 wafer grid
        named("tilt_inversion", inversion(8, 200, 342, 4.5, 10**8)),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _cost(case):
    """Relative cost of a transport: operations, the FP64 path weighted by its slower arithmetic."""
    return work(case)["flops"] * (40 if case["precision"] == 64 else 1)


def draw(rng):
    kind = rng.choice(("transport",) * 6 + ("fit",) * 2 + ("inversion",))
    if kind == "fit":
        while True:
            case = fit(_log_uniform(rng, 16, 65536), rng.choice((342, 342, int(_log_uniform(rng, 25, 1000)))), rng.randint(2, 8))
            if case["B"] * case["J"] * case["K"] <= 32768 * 342 * 4:
                return case
    if kind == "inversion":
        areas = rng.choice((342, int(_log_uniform(rng, 50, 342))))
        return inversion(rng.randint(3, 24), int(_log_uniform(rng, 50, 300)), areas, 4.5, _log_uniform(rng, 1e6, 1e8))
    limit = 0.3 * _cost(transport("sweep", 167342381, chambers=64))
    while True:
        precision = rng.choice((32, 32, 32, 64))
        entry = rng.choice(("run", "run", "once", "noalloc")) if precision == 32 else "run"
        system = rng.choice(("single", "quaternary", "quaternary", "legs", "sweep")) if entry == "run" else "quaternary"
        grid = 50 if system in ("single", "legs") else 200
        case = transport(
            system, _log_uniform(rng, 1e4, 5e5 if precision == 64 else 6e6 if entry == "noalloc" else 3e7),
            pressure=_log_uniform(rng, 0.1, 2.0), tilt=rng.uniform(0.0, 40.0), distance=rng.uniform(80.0, 200.0),
            grid=rng.choice((grid, rng.randint(20, 200))), chambers=rng.randint(2, 24) if system == "sweep" else 1,
            entry=entry, precision=precision, arrivals=rng.random() < 0.25,
            records=rng.random() < 0.25, measured=rng.random() < 0.25, chimneys=system == "quaternary" and rng.random() < 0.25)
        if case["chimneys"]:
            # tubes of 30 mm around the targets stay inside the chamber at the standard place
            case.update(tilt=25.0, distance=150.0)
        if case["records"] and case["n"] > 3_000_000:
            case["records"] = False
        if _cost(case) <= limit:
            return case


# ---------------------------------------------------------------------------------------------------------
# transport
# ---------------------------------------------------------------------------------------------------------
def _shares(n, parts):
    """n atoms split in proportion to parts, at least one each."""
    total = float(sum(parts))
    return [max(1, int(round(n * p / total))) for p in parts]


def _chambers(case):
    """(pressure, tilt, distance, weight) of each chamber of a four-cathode system or sweep: the sweep draws its
    chambers as sputter_inputs.quaternary_sweep does."""
    if case["system"] != "sweep":
        return [(case["pressure"], case["tilt"], case["distance"], 1.0)]
    r = np.random.default_rng(SWEEP_SEED)
    return [(float(r.uniform(0.1, 2.0)), float(r.uniform(0.0, 40.0)), float(r.uniform(80.0, 200.0)), 10.0 ** float(r.uniform(5.0, 7.0)))
            for _ in range(case["chambers"])]


def _configs(case):
    g = case["grid"]
    if case["system"] in ("single", "legs"):
        pressures = (0.5, 0.0, 2.0) if case["system"] == "legs" else (case["pressure"],)
        out = [si.single_ni(p, max(1, case["n"] // len(pressures)), nu=g, nv=g) for p in pressures]
    else:
        cells = _chambers(case)
        counts = _shares(case["n"], [c[3] for c in cells])
        out = [si.quaternary(p, t, d, _shares(n, si.QUAT_POWERS), grid_n=g) for (p, t, d, _), n in zip(cells, counts)]
    if case["measured"]:
        profile = si.measured_racetrack(seed=0)
        out = [si.with_launch(c, profile, si.UNDER_COSINE) for c in out]
    if case["chimneys"]:
        out = [si.with_chimneys(c) for c in out]
    return out


def _history(kind, p):
    if p <= 0.0:
        return 0.0, 0.0, 0.0
    x = math.log(p)
    return tuple(float(np.interp(x, np.log(HISTORY_P), v)) if i != 1 else
                 float(np.exp(np.interp(x, np.log(HISTORY_P), np.log(np.maximum(v, 1e-2))))) for i, v in enumerate(HISTORY[kind]))


def _transport_work(case):
    if case["system"] in ("single", "legs"):
        pressures = (0.5, 0.0, 2.0) if case["system"] == "legs" else (case["pressure"],)
        parts = [("single", p, case["n"] / len(pressures)) for p in pressures]
        bins, segments = case["grid"] ** 2 * len(pressures), len(pressures)
    else:
        cells = _chambers(case)
        total = sum(c[3] for c in cells)
        parts = [("chimneys" if case["chimneys"] else "confocal", c[0], case["n"] * c[3] / total) for c in cells]
        bins, segments = case["grid"] ** 2 * 4 * len(cells), 4 * len(cells)
    ops = 0.0
    for kind, p, n in parts:
        coll, steps, therm = _history(kind, p)
        ops += n * (OPS_LAUNCH + (coll + 1.0 - therm) * OPS_FLIGHT + coll * OPS_COLLISION + (steps + therm) * OPS_STEP)
    out = bins * 16 + segments * 64
    out += 56 * case["n"] if case["records"] else 0
    out += (bins * 8 + segments * 150 * 8) if case["arrivals"] else 0
    return {"bytes": int(out), "flops": int(ops)}


# ---------------------------------------------------------------------------------------------------------
# composition fit
# ---------------------------------------------------------------------------------------------------------
def _fit_inputs(case, seed):
    """Arrival fractions of K cathodes over the areas (a lobe of each cathode on the wafer), rate lines, powers,
    masses, densities, calibration values, and a target library."""
    B, J, K = case["B"], case["J"], case["K"]
    r = np.random.default_rng(seed)
    cen = np.asarray(spx.area_centres(J, 4.5)) / max(1.0, 4.5 * math.sqrt(J / math.pi))
    az = 2.0 * math.pi * np.arange(K) / K
    lobe = cen[:, 0][None, :] * np.cos(az)[:, None] + cen[:, 1][None, :] * np.sin(az)[:, None]
    f = 0.1 * r.uniform(0.6, 1.4, (K, 1)) * np.exp(0.7 * lobe) * (1.0 + 0.01 * r.standard_normal((K, J)))
    a, b = r.uniform(0.5, 2.0, K), r.uniform(0.0, 0.2, K)
    M, rho = r.uniform(50.0, 200.0, K), r.uniform(8.0, 22.0, K)
    P = r.uniform(20.0, 200.0, (B, K))
    Pt = r.uniform(20.0, 200.0, K)
    y = (a * Pt + b)[:, None] * (rho / (M * f.mean(axis=1)))[:, None] * f
    target = (100.0 * y / y.sum(axis=0)).T + 0.3 * r.standard_normal((J, K))
    return [torch.as_tensor(v, dtype=torch.float32, device="cuda").contiguous()
            for v in (f, a, b, P, M, rho, f.mean(axis=1), target)]


def _fit_exact(case, seed):
    *xs, target = [t.double() for t in _fit_inputs(case, seed)]
    xs = [t.requires_grad_(True) for t in xs]
    f, a, b, P, M, rho, fref = xs
    w = (a * P + b) * rho / (M * fref)
    y = w[:, None, :] * f.t()[None]
    c = 100.0 * y / y.sum(dim=2, keepdim=True)
    loss = ((c - target) ** 2).sum(dim=(1, 2))
    return [c.detach(), loss.detach(), *torch.autograd.grad(loss.sum(), xs)]


# ---------------------------------------------------------------------------------------------------------
# tilt inversion
# ---------------------------------------------------------------------------------------------------------
def _tilts(case):
    return [float(v) for v in np.linspace(TILTS[0], TILTS[1], case["T"])]


def _lobes(tilts, grid, n, generator):
    """Deposition profiles [T, 3, grid, grid] of three confocal cathodes as a run of n atoms each tallies them:
    Poisson counts around a lobe whose slope and curvature follow the tilt, over the wafer disc."""
    u = (torch.arange(grid, dtype=torch.float64, device="cuda") + 0.5) * (2.0 / grid) - 1.0
    inside = (u[None, :] ** 2 + u[:, None] ** 2) <= 1.0
    out = torch.empty(len(tilts), 3, grid, grid, dtype=torch.float64, device="cuda")
    area = (100.0 / grid) ** 2
    for t, tilt in enumerate(tilts):
        for k in range(3):
            az = math.pi / 2 * (k + 1)
            s = math.cos(az) * u[None, :] + math.sin(az) * u[:, None]
            p = 0.06 * torch.exp((0.02 * (tilt - 12.0) + 0.35) * s - 0.12 * (u[None, :] ** 2 + u[:, None] ** 2)) / 7854.0
            counts = torch.poisson(p * inside * (n * area), generator=generator)
            out[t, k] = counts / (n * area)
    return out


def _areas64(prof, cen, half_width=2.25):
    """Area means of profiles [..., grid, grid] over squares around the centres, in float64."""
    grid = prof.shape[-1]
    d = 100.0 / grid
    lo = -50.0 + d * torch.arange(grid, dtype=torch.float64, device=prof.device)

    def overlap(c):
        return torch.clamp(torch.minimum(lo + d, c[:, None] + half_width) - torch.maximum(lo, c[:, None] - half_width), min=0.0)
    ou, ov = overlap(cen[:, 0]), overlap(cen[:, 1])
    s = torch.stack([((ov @ p) * ou).sum(dim=1) for p in prof.reshape(-1, grid, grid)])
    return (s / (ov.sum(dim=1) * ou.sum(dim=1))).reshape(*prof.shape[:-2], cen.shape[0])


def _compositions64(f):
    """at.% [T, J, 3] of area values [T, 3, J], each library normalised by the mean of its areas."""
    a, b, P, M, rho = (torch.as_tensor(v, dtype=torch.float64, device=f.device) for v in si.ternary_composition_inputs())
    y = ((a * P + b) * rho / M)[None, :, None] / f.mean(dim=2, keepdim=True) * f
    return (100.0 * y / y.sum(dim=1, keepdim=True)).transpose(1, 2)


def _inversion_inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    prof = _lobes(_tilts(case), case["grid"], case["n"], g)
    cen = torch.as_tensor(spx.area_centres(case["areas"], case["pitch"]), device="cuda")
    measured = _compositions64(_areas64(_lobes([12.7], case["grid"], case["n"], g), cen))[0]
    return prof, cen, measured.float().contiguous()


def _hull_fraction(c):
    """Area of the convex hull of compositions [J, 3] in the ternary diagram over the diagram's."""
    pts = sorted(set(map(tuple, np.stack([c[:, 1] + 0.5 * c[:, 2], c[:, 2] * (math.sqrt(3.0) / 2.0)], axis=1).tolist())))
    if len(pts) < 3:
        return 0.0

    def chain(seq):
        h = []
        for p in seq:
            while len(h) > 1 and (h[-1][0] - h[-2][0]) * (p[1] - h[-2][1]) - (h[-1][1] - h[-2][1]) * (p[0] - h[-2][0]) <= 0.0:
                h.pop()
            h.append(p)
        return h[:-1]
    h = np.asarray(chain(pts) + chain(pts[::-1]))
    x, y = h[:, 0], h[:, 1]
    return 0.5 * float(np.sum(x * np.roll(y, -1) - np.roll(x, -1) * y)) / (math.sqrt(3.0) / 4.0 * 1e4)


def _inversion_exact(case, seed):
    prof, cen, measured = _inversion_inputs(case, seed)
    x = np.asarray(_tilts(case))
    f = _areas64(prof, cen)
    c = _compositions64(f)
    loss = ((c - measured.double()[None]) ** 2).sum(dim=(1, 2))
    u = (x - x.mean()) / (0.5 * (x[-1] - x[0]))
    y = loss.cpu().numpy()
    p2, p1, _ = np.polyfit(u, y, 2)
    vertex = x.mean() - 0.5 * (x[-1] - x[0]) * p1 / (2.0 * p2) if p2 > 0.0 else x[int(np.argmin(y))]
    area = np.array([_hull_fraction(ci) for ci in c.cpu().numpy()])
    area_m = _hull_fraction(measured.double().cpu().numpy())
    slope, offset = np.polyfit(u, area, 1)
    match = x.mean() + 0.5 * (x[-1] - x[0]) * (area_m - offset) / slope
    match = match if x[0] <= match <= x[-1] else math.nan

    def t64(v):
        return torch.as_tensor(np.atleast_1d(v), dtype=torch.float64)
    return dict(f=f, c=c, loss=loss, x_min_de=t64(min(max(vertex, x[0]), x[-1])), area=t64(area), area_measured=t64(area_m),
                x_match_area=t64(match))


# ---------------------------------------------------------------------------------------------------------
# the measured interface
# ---------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    if case["kind"] == "fit":
        *xs, target = _fit_inputs(case, seed)
        return dict(kind="fit", xs=[t.requires_grad_(True) for t in xs], target=target)
    if case["kind"] == "inversion":
        prof, cen, measured = _inversion_inputs(case, seed)
        x = _tilts(case)
        # the plan of the sweep gives the chain its layout; its own runs are not part of this case
        cfgs = [si.ternary(0.5, t, n_particles=1000, grid_n=case["grid"]) for t in x]
        comp = [torch.as_tensor(v, device="cuda") for v in si.ternary_composition_inputs()]
        return dict(kind="inversion", plan=spx.Plan(cfgs, si.Params()), out={"profiles": prof.reshape(-1)}, x=x, comp=comp,
                    measured=measured, centres=cen)
    cfgs = _configs(case)
    state = dict(kind="transport", entry=case["entry"], seed=int(seed), records=case["records"], arrivals=case["arrivals"])
    if case["entry"] == "once":
        return dict(state, cfgs=cfgs, params=si.Params(), precision=case["precision"])
    plan = spx.Plan(cfgs, si.Params(), precision=case["precision"])
    if case["autotune"]:
        plan.autotune()
    state["plan"] = plan
    if case["entry"] == "noalloc":
        state["bufs"] = plan.allocate(records=case["records"], arrivals=case["arrivals"])
    return state


OUTPUTS = ("counts", "counters", "profiles", "records", "arrival_energy", "arrival_angle", "energy_sum")


def run(state):
    if state["kind"] == "fit":
        c = spx.CompositionMap.apply(*state["xs"])
        loss = spx.SquaredDistance.apply(c, state["target"])
        return [c.detach(), loss.detach(), *torch.autograd.grad(loss.sum(), state["xs"])]
    if state["kind"] == "inversion":
        return spx.invert_sweep(state["plan"], state["out"], state["x"], state["comp"], state["measured"], centres=state["centres"])
    if state["entry"] == "noalloc":
        state["plan"].run_noalloc_into(state["seed"], state["bufs"])
        out = state["bufs"]
    elif state["entry"] == "once":
        out = spx.run(state["cfgs"], seed=state["seed"], params=state["params"], precision=state["precision"],
                      records=state["records"], arrivals=state["arrivals"])
    else:
        out = state["plan"].run(seed=state["seed"], records=state["records"], arrivals=state["arrivals"])
    return {k: out[k] for k in OUTPUTS if out.get(k) is not None}


def work(case):
    if case["kind"] == "transport":
        return _transport_work(case)
    if case["kind"] == "fit":
        B, J, K = case["B"], case["J"], case["K"]
        n = B * J * K
        # compositions written once and read by the distance, its gradient written and read: the map, the distance
        # and their backward are separate calls
        small = 4 * (2 * K * J + 10 * K + 2 * B * K + J * K + B)
        return {"bytes": 4 * 5 * n + small, "flops": 30 * n}
    T, g, J = case["T"], case["grid"], case["areas"]
    bins = (4.5 / (100.0 / g) + 1.0) ** 2
    return {"bytes": int(8 * 3 * T * g * g + 3 * T * J * (8 * 2 + 4 * 2)), "flops": int(3 * T * J * (4 * bins + 40))}


def exact(case, seed):
    if case["kind"] == "fit":
        return _fit_exact(case, seed)
    if case["kind"] == "inversion":
        return _inversion_exact(case, seed)
    return None
