"""Timed workloads of the framework, through its public entry points.

``listed()`` names the workloads, ``draw(rng)`` makes more of the same ranges,
``prepare(case, seed)`` builds what a user's program has in hand before the
call (a simulation, batch or server with its mesh, and device-resident initial
counts drawn from the seed), ``run(state)`` makes one pass through the entry
points and returns the counts (and records) it computed, and ``work(case)``
gives the bytes and operations a pass cannot do without.

Each pass starts from the given initial counts again (``set_counts``), so all
passes of a state do the same windows; the outputs are molecule counts, whole
numbers that depend on nothing but the inputs and the seed.  The larger
workloads fix the launch shape the online tuner settles on for them, so that a
pass holds no tuning windows; the smaller ones keep the defaults.
"""
import functools
import math

import numpy as np
import torch

from paper_1610_02258_amd import inputs, rdx

AVOGADRO = 6.02214076e23

# Launch shapes: the library's default, and what the tuner picks where tiles
# cost the same (static ranges) and where they differ (claimed at run time).
SHAPES = {
    "default": None,
    "static": dict(autotune=False, fast_grid_div=1, graph_windows=8, event_group=4, tile_claim=0),
    "claimed": dict(autotune=False, fast_grid_div=1, graph_windows=8, event_group=16, tile_claim=1),
}


def listed():
    return [
        # the smallest call: a 10 ms run of a 1,296-tet box is one window, cut at
        # its end; a program that sweeps parameters makes thousands of them
        dict(name="small_one_window", form="single", model="abc", nx=6, ny=6, nz=6, h_um=1.0, jitter=0.0,
             density=18.5, windows=1, shape="default"),
        # a short trajectory of the same kind on an odd box: launches and their
        # latency, window after window
        dict(name="small_trajectory", form="single", model="chain", nx=7, ny=5, nz=11, h_um=1.0, jitter=0.1,
             density=21.0, windows=101, shape="default"),
        # the simple-model benchmark: 480,000 tets, about two molecules per
        # tet, its whole 100 ms
        dict(name="simple_100ms", form="single", model="simple10", nx=20, ny=20, nz=200, h_um=0.5, jitter=0.1,
             density=100.0, windows=220, shape="static"),
        # the same box at ten times the density (the density series)
        dict(name="simple_dense", form="single", model="simple10", nx=20, ny=20, nz=200, h_um=0.5, jitter=0.1,
             density=1000.0, windows=100, shape="claimed"),
        # the coarse end of the refinement series: 60,000 tets, 17 molecules each
        dict(name="simple_coarse", form="single", model="simple10", nx=10, ny=10, nz=100, h_um=1.0, jitter=0.1,
             density=100.0, windows=100, shape="static"),
        # its fine end: 3.84 million tets, most of them empty
        dict(name="simple_refined", form="single", model="simple10", nx=40, ny=40, nz=400, h_um=0.25, jitter=0.1,
             density=100.0, windows=40, shape="claimed"),
        # the calcium model on the million-tet dendrite: every tet holds
        # hundreds of molecules, two regions, the first 0.46 ms
        dict(name="dendrite", form="single", model="calcium", tets=1_000_000, windows=64, shape="claimed"),
        # production use of a sub-branch: the influx changes between segments
        # and per-region counts are recorded every few windows
        dict(name="branch_recorded", form="recorded", model="calcium", tets=112_000, windows=120, every=5,
             segments=2, shape="claimed"),
        # one record of the dendrite's per-region counts, as a monitoring
        # program takes it between its own windows
        dict(name="region_record", form="record", model="calcium", tets=1_000_000),
        # an ensemble of uneven boxes advanced together (parameter study)
        dict(name="ensemble", form="batch", model="chain", runs=128, tets_lo=1e3, tets_hi=5e4, windows=80,
             shape="claimed"),
        # a small ensemble of tiny runs, the other end of the same use
        dict(name="ensemble_tiny", form="batch", model="chain", runs=48, tets_lo=2e2, tets_hi=1.5e3, windows=64,
             shape="static"),
        # requests of uneven size handed to the server at once
        dict(name="served_burst", form="served", model="simple10", requests=24, tets_lo=1296, tets_hi=5e4,
             windows=60),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _box_dims(rng, tets):
    """A cuboid of about `tets` tets: odd edges, up to ten times longer than wide."""
    cubes = tets / 6.0
    aspect = rng.uniform(1.0, 10.0)
    a = max(1, int(round((cubes / aspect) ** (1.0 / 3.0))))
    b = max(1, a + rng.randint(-a // 4, a // 4))
    return a, b, max(1, int(cubes / (a * b)))


def draw(rng):
    form = rng.choice(["single", "single", "single", "dendrite", "recorded", "record", "batch", "served"])
    shape = rng.choice(["default", "static", "claimed"])
    if form == "single":
        tets = _log_uniform(rng, 1e3, 1.5e6)
        nx, ny, nz = _box_dims(rng, tets)
        per_tet = _log_uniform(rng, 0.2, 25.0)  # molecules per tet
        h = _log_uniform(rng, 0.25, 1.0)
        windows = max(1, min(240, int(_log_uniform(rng, 1.0, 240.0)), int(6e7 / (tets * (1.0 + 0.2 * per_tet)))))
        return dict(form="single", model=rng.choice(["abc", "chain", "simple10"]), nx=nx, ny=ny, nz=nz, h_um=h,
                    jitter=rng.choice([0.0, 0.1]), density=per_tet * 6.0 / h ** 3, windows=windows, shape=shape)
    if form == "dendrite":
        tets = _log_uniform(rng, 3e4, 1e6)
        windows = max(1, min(int(_log_uniform(rng, 8.0, 200.0)), int(6e7 / tets)))
        return dict(form="single", model="calcium", tets=int(tets), windows=windows, shape=shape)
    if form == "recorded":
        every, segments = rng.randint(1, 12), rng.randint(1, 3)
        return dict(form="recorded", model="calcium", tets=int(_log_uniform(rng, 3e4, 3e5)),
                    windows=rng.randint(segments * every, 140), every=every, segments=segments, shape=shape)
    if form == "record":
        return dict(form="record", model="calcium", tets=int(_log_uniform(rng, 3e4, 1e6)))
    if form == "batch":
        runs = int(_log_uniform(rng, 2, 140))
        lo = _log_uniform(rng, 2e2, 2e3)
        return dict(form="batch", model="chain", runs=runs, tets_lo=lo, tets_hi=lo * rng.uniform(2.0, 25.0),
                    windows=rng.randint(8, 80), shape=shape)
    lo = _log_uniform(rng, 1e3, 5e3)
    return dict(form="served", model="simple10", requests=rng.randint(4, 24), tets_lo=lo,
                tets_hi=lo * rng.uniform(1.5, 10.0), windows=rng.randint(8, 60))


# ------------------------------------------------------------------ inputs ----
# Meshes do not depend on the seed: a program keeps its mesh and runs it with
# many seeds and initial counts.

@functools.lru_cache(maxsize=4)
def _box(nx, ny, nz, h_um, jitter):
    return _with_volumes(inputs.box_mesh(nx, ny, nz, h_um * inputs.UM, jitter=jitter, seed=1))


@functools.lru_cache(maxsize=2)
def _dendrite(tets):
    return _with_volumes(inputs.dendrite_mesh(target_tets=tets, seed=2))


def _with_volumes(mesh):
    mesh.volumes = torch.from_numpy(inputs.tet_volumes_for_sampling(mesh))  # m^3
    return mesh


@functools.lru_cache(maxsize=None)
def _uneven_boxes(runs, lo, hi):
    """The cuboids of an ensemble: 6 x 6 x n cubes, sizes uniform over their logarithm."""
    rng = np.random.default_rng(runs)
    return [_box_plain(max(1, int(round(t / 216.0)))) for t in np.exp(rng.uniform(math.log(lo), math.log(hi), runs))]


@functools.lru_cache(maxsize=None)
def _box_plain(n):
    return _with_volumes(inputs.box_mesh(6, 6, n, 1.0 * inputs.UM))


@functools.lru_cache(maxsize=None)
def _model(name):
    return {"abc": inputs.model_abc, "chain": inputs.model_abc_chain, "simple10": inputs.model_simple10,
            "calcium": inputs.model_calcium}[name]()


def _tet_counts(case):
    """Tets of each run of the case (for the work it takes; a dendrite's mesh is built to about `tets`)."""
    if case["form"] in ("batch", "served"):
        runs = case.get("runs") or case["requests"]
        return [m.n_tets for m in _uneven_boxes(runs, case["tets_lo"], case["tets_hi"])]
    return [case["tets"] if "tets" in case else 6 * case["nx"] * case["ny"] * case["nz"]]


def _mean_per_volume(case, model):
    """Mean molecules of each species per m^3."""
    if case["model"] == "calcium":
        return [inputs.CALCIUM_CONC[s] * AVOGADRO * 1e3 for s in model.species]
    density = case.get("density", 25.0) * 1e18  # molecules per um^3
    if case["model"] == "abc":
        return [0.5 * density, 0.5 * density, 0.0]
    if case["model"] == "chain":
        return [0.4 * density, 0.4 * density, 0.0, 0.2 * density, 0.0, 0.0]
    w = np.random.default_rng(101).uniform(0.5, 1.5, model.S)
    return list(density * w / w.sum())


def _counts(mesh, per_volume, gen):
    """Molecules placed uniformly in space: Poisson counts with means proportional to the tets' volumes."""
    rate = torch.tensor(per_volume, dtype=torch.float64)[:, None] * mesh.volumes[None, :]
    return torch.poisson(rate.cuda(), generator=gen).to(torch.int32).contiguous()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    model = _model(case["model"])
    per_volume = _mean_per_volume(case, model)
    form = case["form"]
    if form == "batch":
        rng = np.random.default_rng(seed)
        meshes = _uneven_boxes(case["runs"], case["tets_lo"], case["tets_hi"])
        runs = [(m.as_dict(), inputs.model_abc_chain(rng.uniform(0.5, 1.5, 4)).as_dict(), seed * 1009 + i)
                for i, m in enumerate(meshes)]
        batch = rdx.Batch(runs)
        batch.set_exec_options(**(SHAPES[case["shape"]] or {}))
        counts = [_counts(m, per_volume, gen) for m in meshes]
        # every run's counts end in one buffer
        out = torch.zeros(sum(c.numel() for c in counts), dtype=torch.int32, device="cuda")
        views = [v.view(c.shape) for v, c in zip(out.split([c.numel() for c in counts]), counts)]
        return dict(form=form, batch=batch, counts=counts, out=out, views=views, windows=case["windows"])
    if form == "served":
        meshes = _uneven_boxes(case["requests"], case["tets_lo"], case["tets_hi"])
        server = rdx.Server(model.as_dict(), 1 << 30)
        tau = rdx.setup_geometry(meshes[0].as_dict(), model.as_dict())["tau"]
        requests = [(m.as_dict(), model.as_dict(), seed * 1009 + i, _counts(m, per_volume, gen).cpu().numpy())
                    for i, m in enumerate(meshes)]
        return dict(form=form, server=server, requests=requests, t_end=(case["windows"] - 0.5) * tau)
    mesh = _dendrite(case["tets"]) if "tets" in case else _box(*(case[k] for k in ("nx", "ny", "nz", "h_um", "jitter")))
    sim = rdx.Sim(mesh.as_dict(), model.as_dict(), seed)
    if case.get("shape") and SHAPES[case["shape"]]:
        sim.set_exec_options(**SHAPES[case["shape"]])
    counts = _counts(mesh, per_volume, gen)
    state = dict(form=form, sim=sim, counts=counts, out=torch.empty_like(counts))
    if form == "single":
        # the end time falls inside the last window, which is cut there
        state["t_end"] = (case["windows"] - 0.5) * sim.tau
    elif form == "record":
        sim.set_counts(counts)
        state["sums"] = torch.empty((sim.n_regions, sim.S), dtype=torch.int64, device="cuda")
    else:
        rng = np.random.default_rng(seed)
        base = np.asarray(model.as_dict()["kcst"])
        per_segment = case["windows"] // case["segments"]
        state["per_segment"], state["every"] = per_segment, case["every"]
        state["rates"] = []
        for _ in range(case["segments"]):  # the influx (order 0) is redrawn for each segment
            k = base.copy()
            k[1, 18] *= rng.uniform(0.5, 3.0)
            state["rates"].append(k)
        slots = max(1, per_segment // case["every"])
        state["rings"] = torch.zeros((case["segments"], slots, sim.n_regions, sim.S), dtype=torch.int64, device="cuda")
    return state


def run(state):
    form = state["form"]
    if form == "single":
        sim = state["sim"]
        sim.set_counts(state["counts"])
        sim.run(state["t_end"])
        return sim.get_counts(out=state["out"])
    if form == "record":
        return state["sim"].region_counts(out=state["sums"])
    if form == "recorded":
        sim = state["sim"]
        sim.set_counts(state["counts"])
        for kcst, ring in zip(state["rates"], state["rings"]):
            sim.set_rate_constants(kcst)
            sim.step_recorded(state["per_segment"], state["every"], ring)
        return [sim.get_counts(out=state["out"]), state["rings"]]
    if form == "batch":
        batch = state["batch"]
        batch.set_counts_all(state["counts"])
        batch.step(state["windows"])
        for i, view in enumerate(state["views"]):
            batch.get_counts(i, out=view)
        return state["out"]
    server = state["server"]
    tickets = [server.submit(mesh, model, seed, counts, state["t_end"])
               for mesh, model, seed, counts in state["requests"]]
    return [server.wait(t)[0] for t in tickets]


def exact(case, seed):
    """Every output is a molecule count, a whole number: no 64-bit value stands behind it."""
    return None


def work(case):
    """Bytes: the counts in and out of a pass; and for each window, whose moves
    reach across the whole mesh, the counts read and written and the mesh's
    neighbours, couplings and volumes read (8 S + 56 bytes a tet).  Operations:
    the random words of a window, one Philox call (60 integer operations) for
    each four words, one word per molecule of a small count and a few per face
    of a large one."""
    model = _model(case["model"])
    tets = _tet_counts(case)
    T, S = sum(tets), model.S
    if case["form"] == "record":
        return dict(bytes=T * (4 * S + 1), flops=T * S)
    windows = case["windows"]
    if case["model"] == "calcium":
        volume = 1.783e-15 / case["tets"]  # m^3 of the dendrite, by tet
        per_tet = [c * volume for c in _mean_per_volume(case, model)]
    else:
        h = case.get("h_um", 1.0) * inputs.UM
        per_tet = [c * h ** 3 / 6.0 for c in _mean_per_volume(case, model)]
    words = sum(n if n <= 16.0 else 4.0 for n in per_tet)
    return dict(bytes=8 * S * T + windows * T * (8 * S + 56), flops=float(windows * T * words * 15.0))
