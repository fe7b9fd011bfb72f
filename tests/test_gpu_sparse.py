"""Batches of sparse realizations (a hash table of occupied pairs in LDS, one
block per realization) against the oracle: tets in such number for the SSA
that the block sorts out those without an event, reactions of a species with
itself, reaction regions, the method's options, a species that does not move,
and more species than one look-up takes.  Every count after every run."""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def note(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    import paper_1512_03126_amd as mod

    mod.lib()
    return mod


# a realization does not fit a compute unit, or not with another, and there are more of them than units
WIDE, SMALL, SMALLEST = (13, 13, 14), (8, 8, 8), (6, 6, 6)
SEVEN = [([0, 5], [6], 4e8), ([6], [0, 5], 500.0), ([4, 4], [1], 4e8), ([1, 2], [3, 4], 4e8), ([3], [2], 300.0),
         ([2, 6], [5, 5, 1], 4e8), ([5, 6], [0, 3], 3e8), ([0], [4], 200.0), ([1, 1], [0, 2], 3e8)]
SIXTEEN = [([q % 16, (5 * q + 1) % 16], [(3 * q + 2) % 16], 2e8) if q % 3 else ([q % 16], [(q + 7) % 16, (q + 2) % 16], 90.0)
           for q in range(32)]

CASES = {
    "many tets for the SSA": dict(cells=WIDE, S=3, rx=[([0], [1], 300.0), ([1], [0], 200.0), ([0, 2], [1], 1e8)],
                                  molecules=1000),
    "pairs of one species": dict(cells=WIDE, S=3, rx=[([0, 0], [1], 4e8), ([1], [0, 0], 900.0), ([2, 2], [0, 1], 4e8)],
                                 molecules=400, together=3),
    "regions": dict(cells=WIDE, S=2, rx=[([0, 1], [1], 2e9), ([0], [0, 1], 200.0), ([1], [], 400.0)], molecules=500,
                    regions={0: 3, 1: 5, 2: 2}),
    "first-order means, sequential splits from two": dict(
        cells=WIDE, S=3, rx=[([0, 1], [2], 2e9), ([2], [0, 1], 900.0)], molecules=400, together=4,
        method=dict(occupancy_correction=False, split_threshold=2)),
    "seven species": dict(cells=SMALL, S=7, rx=SEVEN, molecules=60, together=2),
    "seven species, second transfer form": dict(cells=SMALL, S=7, rx=SEVEN, molecules=60, together=2,
                                                method=dict(transfer_form=1)),
    "seven species without reactions": dict(cells=SMALL, S=7, rx=[], molecules=70),
    "most species and reactions": dict(cells=SMALLEST, S=16, rx=SIXTEEN, molecules=16),
}


@pytest.mark.parametrize("name", list(CASES))
def test_sparse_batch(P, orc, name):
    c = CASES[name]
    S, Rz, seed = c["S"], 300, 17
    xyz, tets = W.kuhn_box(*c["cells"], 0.2e-6)
    T = tets.shape[0]
    note(f"sparse batch: {name}, {Rz} realizations of {T} tets, {S} species, {len(c['rx'])} reactions")
    D = [1e-12 * (0.3 + 0.1 * s) for s in range(S)]
    if S > 2:
        D[2] = 0.0
    regions = {q: np.arange(0, T, every, dtype=np.int32) for q, every in c.get("regions", {}).items()}
    method = c.get("method", {})
    g = P.Simulation(xyz, tets, D, c["rx"], seed=seed, n_realizations=Rz, regions=regions, **method)
    e = P.rdos_engine_create(0, 0)

    def request(n):
        t = P.rdos_engine_submit(e, g.h, n, 1.0)
        P.rdos_engine_drain(e)
        P.rdos_engine_release(e, t)

    if c["cells"] == WIDE:
        request(331)  # empty: the queue is tuned for lists of this size first
    rng = np.random.default_rng(seed)
    together = c.get("together", 1)  # molecules placed at a time
    refs = {}
    for r in range(Rz):
        init = np.stack([together * np.bincount(rng.integers(0, T, c["molecules"] // together), minlength=T)
                         for _ in range(S)]).astype(np.int32)
        for s in range(S):
            g.set_counts(s, init[s], realization=r)
        if r in (0, Rz - 1):
            o = orc.OracleSim(xyz, tets, D, c["rx"], seed=seed, realization=r)
            if method.get("transfer_form"):
                o.set_transfer_form(1)
            if "occupancy_correction" in method:
                o.set_first_order(True)
            if "split_threshold" in method:
                o.set_split_threshold(method["split_threshold"])
            for q, where in regions.items():
                o.set_reaction_region(q, where)
            for s in range(S):
                o.set_counts(s, init[s])
            t, k = g.time()
            o.set_state(k, t)
            refs[r] = o
    for n in (8, 33, 15):
        request(n)
        for r, o in refs.items():
            o.run_steps(n)
            got, want = g.get_counts(None, realization=r), o.get_counts()
            assert np.array_equal(got, want), (name, n, r, int((got != want).sum()))
    P.rdos_engine_destroy(e)
    g.close()
