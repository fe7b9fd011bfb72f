"""The work that a user of this framework has it do, as cases to be measured.

Each case is one pass through the public entry points: stepping one
simulation or an ensemble of realizations and reading the counts, a batch of
simulations through the engine, requests served whole (mesh in, counts out),
or setting up a mesh.  Sizes are those of the repository's own workloads,
tests and benchmark, of the paper's cylinder, and odd ones between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1512_03126_amd as P
import workloads as W

# ----------------------------------------------------------------------------
# Cases
# ----------------------------------------------------------------------------
_BASE = {"path": "step", "mesh": "box", "nx": 5, "ny": 5, "nz": 5, "edge_um": 0.2, "jitter": False,
         "chem": "diffusion", "mean": 1.0, "place": "uniform", "realizations": 1, "nx2": 0, "realizations2": 0,
         "periods": 1, "form": 0, "read": "host"}


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: the 1 um cube sampled after every period, as for a time trace.
        _case(name="cube_sample", mean=1000 / 750, place="point"),
        # The same cube run over the 0.5 s of the paper's example (422 full periods), then read.
        _case(name="cube_run", mean=1000 / 750, place="point", periods=422),
        # The paper's performance model: about 1060 tets, 1e5 molecules placed uniformly, diffusion only.
        _case(name="bar_uniform", nx=20, ny=3, nz=3, edge_um=0.5, mean=1e5 / 1080, periods=100),
        # The paper's reaction-diffusion performance model: 10 species, 8 reactions, 0.1 to 1 uM.
        _case(name="bar_ten", nx=20, ny=3, nz=3, edge_um=0.5, chem="ten", mean=5.0, periods=100),
        # A validation ensemble (production and pair annihilation on the cube): many realizations of a small
        # mesh, a reaction without reactants in every tet.
        _case(name="ensemble_birth", chem="birth", mean=30 / 750, realizations=1000, periods=169, read="device"),
        # One realization of the 384,000-tet A+B<->C system over its whole 0.1 s.
        _case(name="abc_384k", nx=40, ny=40, nz=40, edge_um=0.1, chem="abc", mean=0.01, periods=338),
        # The jittered lattice with a fourth species, many short periods.
        _case(name="jitter_384k", nx=40, ny=40, nz=40, edge_um=0.1, jitter=True, chem="abcd", mean=0.02, periods=200),
        # A crowded volume: every tet holds tens of molecules of each species and fires reactions each period.
        _case(name="crowded_162k", nx=30, ny=30, nz=30, edge_um=0.1, chem="abc_fast", mean=30.0, periods=20),
        # The benchmark's batch: 256 realizations of 384,000 tets and 64 of 48,000 through the engine.
        _case(name="batched_mix", path="engine", nx=40, ny=40, nz=40, edge_um=0.1, chem="abc", mean=0.01,
              realizations=256, nx2=20, realizations2=64, periods=338, read="device"),
        # Surface diffusion and reactions, the split-at-once transfer form, a medium ensemble.
        _case(name="surface_form1", path="engine", mesh="surface", nx=200, ny=201, nz=1, edge_um=0.1,
              chem="abc_surface", mean=0.05, realizations=16, periods=200, form=1, read="device"),
        # Served requests, whole: mesh, model and counts on the host in, counts out.
        {"name": "serve_mix", "path": "serve", "cells": "12,21,34,55", "species": "1,6,3,4", "model": 11,
         "periods": 1000},
        # Setting up a mesh of a million tets (a moved lattice) and reading its tables.
        {"name": "setup_1m", "path": "setup", "cells": "55"},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(_log_uniform(rng, lo, hi)))))


def draw(rng):
    kind = rng.choice(["cube", "bar", "ten", "ensemble", "plain", "jitter", "crowded", "batch", "surface", "serve",
                       "setup"])
    if kind == "cube":
        n = rng.randint(3, 7)
        return _case(nx=n, ny=n, nz=rng.randint(3, 7), mean=_log_uniform(rng, 0.1, 5.0),
                     place=rng.choice(["point", "uniform"]), periods=_log_int(rng, 1, 500))
    if kind == "bar":
        return _case(nx=rng.randint(8, 41), ny=rng.randint(2, 4), nz=rng.randint(2, 4), edge_um=0.5,
                     mean=_log_uniform(rng, 1.0, 200.0), periods=_log_int(rng, 10, 200))
    if kind == "ten":
        return _case(nx=rng.randint(8, 31), ny=rng.randint(2, 4), nz=rng.randint(2, 4), edge_um=0.5, chem="ten",
                     mean=_log_uniform(rng, 0.5, 12.0), periods=_log_int(rng, 10, 200))
    if kind == "ensemble":
        return _case(nx=rng.randint(3, 9), ny=rng.randint(3, 6), nz=rng.randint(3, 6),
                     chem=rng.choice(["birth", "abc_fast"]), mean=_log_uniform(rng, 0.02, 2.0),
                     realizations=_log_int(rng, 24, 1500), periods=_log_int(rng, 10, 169), read="device")
    if kind == "plain":
        return _case(nx=rng.randint(12, 40), ny=rng.randint(12, 40), nz=rng.randint(12, 40), edge_um=0.1, chem="abc",
                     mean=_log_uniform(rng, 0.003, 0.3), periods=_log_int(rng, 30, 338))
    if kind == "jitter":
        n = rng.randint(12, 40)
        return _case(nx=n, ny=n, nz=n, edge_um=0.1, jitter=True, chem="abcd", mean=_log_uniform(rng, 0.005, 0.1),
                     periods=_log_int(rng, 30, 300), form=rng.randint(0, 1))
    if kind == "crowded":
        return _case(nx=rng.randint(8, 30), ny=rng.randint(8, 30), nz=rng.randint(8, 30), edge_um=0.1,
                     chem="abc_fast", mean=_log_uniform(rng, 1.0, 60.0), periods=_log_int(rng, 5, 20))
    if kind == "batch":
        n = rng.randint(15, 40)
        return _case(path="engine", nx=n, ny=n, nz=n, edge_um=0.1, chem=rng.choice(["abc", "abc", "abcd"]),
                     mean=_log_uniform(rng, 0.003, 0.03), realizations=_log_int(rng, 24, 128), nx2=rng.randint(6, 20),
                     realizations2=_log_int(rng, 1, 64), periods=_log_int(rng, 60, 338), read="device")
    if kind == "surface":
        return _case(path="engine", mesh="surface", nx=rng.randint(60, 300), ny=rng.randint(60, 300), nz=1,
                     edge_um=0.1, chem="abc_surface", mean=_log_uniform(rng, 0.01, 0.3),
                     realizations=_log_int(rng, 1, 32), periods=_log_int(rng, 50, 250), form=rng.randint(0, 1),
                     read="device")
    if kind == "serve":
        k = rng.randint(1, 4)
        return {"path": "serve", "cells": ",".join(str(_log_int(rng, 12, 55)) for _ in range(k)),
                "species": ",".join(str(rng.randint(1, 6)) for _ in range(k)), "model": rng.randint(1, 10**6),
                "periods": _log_int(rng, 300, 1000)}
    return {"path": "setup", "cells": str(_log_int(rng, 8, 55))}


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------
def _mesh(nx, ny, nz, c, seed):
    a = c["edge_um"] * 1e-6
    if c["mesh"] == "surface":
        return W.triangle_lattice(nx, ny, a)
    xyz, tets = W.kuhn_box(nx, ny, nz, a)
    if c["jitter"]:
        xyz = W.jitter(xyz, nx, a, 0.2, seed)
    return xyz, tets


def _chemistry(c, n_cells):
    """(diffusion coefficients, reactions, mean molecules per tet and species)."""
    a = c["edge_um"] * 1e-6
    m = c["mean"]
    if c["chem"] == "diffusion":
        return [1e-12], [], [m]
    if c["chem"] == "abc":
        return [1e-12, 1e-12, 0.5e-12], [([0, 1], [2], 1e6), ([2], [0, 1], 10.0)], [m, m, 0.0]
    if c["chem"] == "abc_fast":
        return [1e-12, 1e-12, 0.5e-12], [([0, 1], [2], 1e6), ([2], [0, 1], 1000.0)], [m, m, 0.1 * m]
    if c["chem"] == "abcd":
        return ([1e-12, 1e-12, 0.5e-12, 5e-12],
                [([0, 1], [2], 1e6), ([2], [0, 1], 10.0), ([3], [], 0.01)], [m, m, 0.0, 2 * m])
    if c["chem"] == "abc_surface":
        k2 = 10.0 * W.N_A * 0.5 * a * a  # 10 /s per pair in one triangle
        return [1e-12, 1e-12, 0.5e-12], [([0, 1], [2], k2), ([2], [0, 1], 10.0)], [m, m, 0.0]
    if c["chem"] == "birth":
        # 0 -> A and A + A -> 0 with the well-mixed mean at `mean` per tet
        nav = W.N_A * 1e3 * n_cells * a ** 3 / 6.0
        mu = 1e8 / nav
        total = m * n_cells
        return [1e-11], [([], [0], 2.0 * mu * total * total / nav), ([0, 0], [], 1e8)], [m]
    chem = W.ten_species(nx=2, ny=1, nz=1, seed=1)
    return list(chem.D), list(chem.reactions), [m * (0.5 + 0.1 * s) for s in range(10)]


def _place(rng, T, mean, how):
    total = int(round(mean * T))
    if how == "point":
        out = np.zeros(T, np.int32)
        out[T // 2] = total
        return out
    if mean >= 0.5:
        return rng.poisson(mean, T).astype(np.int32)
    return np.bincount(rng.integers(0, T, total), minlength=T).astype(np.int32)


def _simulation(c, nx, ny, nz, realizations, seed):
    rng = np.random.default_rng([seed, nx, realizations])
    xyz, tets = _mesh(nx, ny, nz, c, seed)
    T = tets.shape[0]
    D, reactions, means = _chemistry(c, T)
    sim = P.Simulation(xyz, tets, D, reactions, seed=seed, n_realizations=realizations, transfer_form=c["form"])
    for r in range(realizations):
        for s, mean in enumerate(means):
            if mean > 0:
                sim.set_counts(s, _place(rng, T, mean, c["place"]), realization=r)
    return sim


def _request(n, n_species, model, seed):
    """One served request: a jittered lattice with a random chemistry (the
    distributions of the serving workload), its counts on the host."""
    chem = np.random.default_rng([model, n, n_species])
    rng = np.random.default_rng([seed, n, n_species])
    a = 0.1e-6
    xyz, tets = W.kuhn_lattice(n, a)
    xyz = W.jitter(xyz, n, a, 0.2, seed)

    def log_u(lo, hi):
        return float(math.exp(chem.uniform(math.log(lo), math.log(hi))))

    D = [log_u(1e-13, 1e-11) for _ in range(n_species)]
    reactions = []
    for _ in range(int(chem.integers(0, 2 * n_species + 1))):
        if chem.random() < 0.5:
            reac, k = [int(chem.integers(0, n_species))], log_u(1.0, 1e3)
        else:
            reac, k = [int(chem.integers(0, n_species)) for _ in range(2)], log_u(1e5, 1e8)
        prod = [int(chem.integers(0, n_species)) for _ in range(int(chem.integers(0, len(reac) + 1)))]
        reactions.append((reac, prod, k))
    T = tets.shape[0]
    counts = []
    for _ in range(n_species):
        total = W.count_for(log_u(10e-9, 1e-6), (n * a) ** 3)
        counts.append(np.bincount(rng.integers(0, T, total), minlength=T).astype(np.int32))
    return {"xyz": xyz, "tets": tets, "D": D, "reactions": reactions, "counts": counts, "seed": seed}


def _cells(case):
    return [int(x) for x in case["cells"].split(",")]


class _State:
    """What a user's program holds between passes."""

    def __init__(self, case):
        self.case = case
        self.sims, self.engine, self.requests, self.stream = [], None, [], None

    def __del__(self):
        if self.engine is not None:
            P.rdos_engine_destroy(self.engine)
        for s in self.sims:
            s.close()


def prepare(case, seed):
    st = _State(case)
    if case["path"] == "setup":
        n = _cells(case)[0]
        xyz, st.tets = W.kuhn_lattice(n, 0.1e-6)
        st.xyz = W.jitter(xyz, n, 0.1e-6, 0.2, seed)
        return st
    if case["path"] == "serve":
        st.requests = [_request(n, int(s), case["model"], seed)
                       for n, s in zip(_cells(case), case["species"].split(","))]
        st.engine = P.rdos_engine_create(0, 0)
        return st
    st.sims.append(_simulation(case, case["nx"], case["ny"], case["nz"], case["realizations"], seed))
    if case["realizations2"]:
        n = case["nx2"]
        st.sims.append(_simulation(case, n, n, n, case["realizations2"], seed + 1))
    if case["path"] == "engine":
        st.engine = P.rdos_engine_create(0, 0)
    elif case["read"] == "device":
        st.stream = torch.cuda.Stream()
        st.sims[0].set_stream(st.stream)
    return st


# ----------------------------------------------------------------------------
# One pass
# ----------------------------------------------------------------------------
def _read_device(sim):
    """Every realization's and species' counts as one tensor, from the zero-copy views."""
    rows = [sim.device_counts(s, r) for r in range(sim.Rz) for s in range(sim.S)]
    return torch.stack(rows)


def _run_engine(engine, sims, periods):
    P.rdos_engine_hold(engine, True)
    tickets = [P.rdos_engine_submit(engine, s.h, periods, 1.0) for s in sims]
    P.rdos_engine_hold(engine, False)
    P.rdos_engine_drain(engine)
    for t in tickets:
        P.rdos_engine_release(engine, t)


def run(state):
    case = state.case
    if case["path"] == "setup":
        sim = P.Simulation(state.xyz, state.tets, [1e-12, 5e-12])
        out = sim.geometry()
        out["tau"] = sim.tau
        sim.close()
        return out
    if case["path"] == "serve":
        sims = []
        for q in state.requests:
            s = P.Simulation(q["xyz"], q["tets"], q["D"], q["reactions"], seed=q["seed"], tau_scale=None)
            for m, counts in enumerate(q["counts"]):
                s.set_counts(m, counts)
            sims.append(s)
        tickets = [P.rdos_engine_submit(state.engine, s.h, case["periods"], 1.0) for s in sims]
        P.rdos_engine_drain(state.engine)
        out = []
        for t, s in zip(tickets, sims):
            P.rdos_engine_release(state.engine, t)
            out.append(s.get_counts())
            s.close()
        return out
    if case["path"] == "engine":
        _run_engine(state.engine, state.sims, case["periods"])
        out = [_read_device(s) for s in state.sims]
        torch.cuda.current_stream().synchronize()  # the engine's streams may write the counts again after this
        return out
    sim = state.sims[0]
    sim.step(case["periods"])
    if case["read"] == "device":
        with torch.cuda.stream(state.stream):
            return _read_device(sim)
    return [sim.get_counts(None, realization=r) for r in range(sim.Rz)]


# ----------------------------------------------------------------------------
# What a pass cannot do without
# ----------------------------------------------------------------------------
def _period_work(c, cells, realizations):
    """Per period: each tet-species that holds molecules read and written
    once (8 bytes), the 64-byte record of each tet that some realization
    occupies read once; per such tet-species one block of ten Philox rounds
    and the binomial and split in 64-bit arithmetic (about 200 operations)."""
    _, _, means = _chemistry(c, cells)
    held = sum(1.0 - math.exp(-m) for m in means)
    tet = 1.0 - math.exp(-realizations * sum(means))
    n = realizations * cells * held
    return 8.0 * n + 64.0 * cells * tet, 200.0 * n


def work(case):
    if case["path"] == "setup":
        T, nv = 6.0 * _cells(case)[0] ** 3, (_cells(case)[0] + 1.0) ** 3
        return {"bytes": 24.0 * nv + 16.0 * T + 64.0 * T, "flops": 300.0 * T}
    if case["path"] == "serve":
        nbytes = flops = 0.0
        for n, s in zip(_cells(case), case["species"].split(",")):
            T, nv = 6.0 * n ** 3, (n + 1.0) ** 3
            held = 1.0 - math.exp(-0.01)  # 100 nM, the middle of the range, in a tet of 0.1 um cells
            nbytes += 24.0 * nv + 16.0 * T + 64.0 * T + 8.0 * T * int(s)
            nbytes += case["periods"] * T * int(s) * held * (8.0 + 64.0)
            flops += case["periods"] * T * int(s) * held * 200.0
        return {"bytes": nbytes, "flops": flops}
    per_cell = 2 if case["mesh"] == "surface" else 6
    b, f = _period_work(case, per_cell * case["nx"] * case["ny"] * case["nz"], case["realizations"])
    if case["realizations2"]:
        b2, f2 = _period_work(case, per_cell * case["nx2"] ** 3, case["realizations2"])
        b, f = b + b2, f + f2
    return {"bytes": case["periods"] * b, "flops": case["periods"] * f}


# ----------------------------------------------------------------------------
# Values in 64 bits
# ----------------------------------------------------------------------------
def exact(case, seed):
    """The mesh tables from their definition.  Counts are whole numbers drawn
    at random: they have no other value than the one the streams give."""
    if case["path"] != "setup":
        return None
    n, a = _cells(case)[0], 0.1e-6
    xyz, tets = W.kuhn_lattice(n, a)
    xyz = W.jitter(xyz, n, a, 0.2, seed)
    T = tets.shape[0]
    p = xyz[tets]
    e = p[:, 1:] - p[:, :1]
    vol = np.abs(np.einsum("ij,ij->i", np.cross(e[:, 0], e[:, 1]), e[:, 2])) / 6.0
    centre = p.mean(axis=1)
    local = [[1, 2, 3], [0, 2, 3], [0, 1, 3], [0, 1, 2]]
    ids = np.concatenate([np.sort(tets[:, f], axis=1) for f in local]).astype(np.int64)
    nv = xyz.shape[0]
    key = (ids[:, 0] * nv + ids[:, 1]) * nv + ids[:, 2]
    order = np.argsort(key, kind="stable")
    same = np.nonzero(key[order][1:] == key[order][:-1])[0]
    one, two = order[same], order[same + 1]
    nbr = np.full(4 * T, -1, np.int64)
    nbr[one], nbr[two] = two % T, one % T
    nbr = nbr.reshape(4, T).T
    rate = np.zeros((T, 4))
    for f in range(4):
        q = p[:, local[f]]
        area = 0.5 * np.linalg.norm(np.cross(q[:, 1] - q[:, 0], q[:, 2] - q[:, 0]), axis=1)
        delta = np.linalg.norm(centre[nbr[:, f]] - centre, axis=1)
        rate[:, f] = np.where(nbr[:, f] >= 0, area / (vol * np.where(nbr[:, f] >= 0, delta, 1.0)), 0.0)
    g = rate.sum(axis=1)
    return {"nbr": None, "w": rate / g[:, None], "g": g, "nav": W.N_A * vol * 1e3, "tau": float(1.0 / (5e-12 * g.max()))}
