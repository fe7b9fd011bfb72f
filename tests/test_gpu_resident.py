"""Periods with the state held in LDS (one block per realization, or several
that exchange molecules) against the oracle, every count: sizes at the edges
of the cut (16 tets per block, a last block of a few tets, one block, more
realizations than blocks fit), every species and reaction bound of the lane
state, odd and even runs, and runs that alternate with the other launch
paths, which must find the counts, the empty buffer and the occupancy bytes
as they leave them."""
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


def chemistry(S, R):
    """S species, R reactions of every order: bindings, decays, pair
    annihilations and (from four reactions on) a production."""
    D = [1e-12 * (0.3 + 0.2 * s) for s in range(S)]
    D[S // 2] = 0.0 if S > 2 else D[S // 2]
    rx = []
    for q in range(R):
        a, b, c = q % S, (q + 1) % S, (q + 2) % S
        kind = q % 4
        if kind == 0 and S > 1:
            rx.append(([a, b], [c], 2e8))
        elif kind == 1:
            rx.append(([a], [b, c], 60.0))
        elif kind == 2:
            rx.append(([a, a], [b], 1e8))
        else:
            rx.append(([], [a], 2e-4))
    return D, rx


def both(P, orc, shape, S, R, Rz, mean, seed=5, crowded=None, **method):
    xyz, tets = W.kuhn_box(*shape, 0.2e-6)
    T = tets.shape[0]
    D, rx = chemistry(S, R)
    rng = np.random.default_rng(seed)
    init = rng.poisson(mean, (Rz, S, T)).astype(np.int32)
    if crowded is None:
        init[:, 0, ::11] += 12
    else:
        init[:, :, int(crowded * T):] = 0
    g = P.Simulation(xyz, tets, D, rx, seed=seed, n_realizations=Rz, **method)
    refs = {}
    for r in range(Rz):
        for s in range(S):
            g.set_counts(s, init[r, s], realization=r)
    for r in sorted({0, Rz // 2, Rz - 1}):
        o = orc.OracleSim(xyz, tets, D, rx, seed=seed, realization=r)
        for s in range(S):
            o.set_counts(s, init[r, s])
        refs[r] = o
    return g, refs


def check(g, refs, what):
    for r, o in refs.items():
        got, want = g.get_counts(None, realization=r), o.get_counts()
        assert np.array_equal(got, want), (what, r, int((got != want).sum()))


@pytest.mark.parametrize("shape,S,R,Rz,mean", [
    ((1, 1, 1), 1, 0, 1, 3.0),      # 6 tets: one block of less than a wavefront
    ((1, 1, 3), 2, 2, 1, 3.0),      # 18 tets: a second block of 2 tets
    ((2, 2, 2), 3, 3, 1, 2.0),      # 48 tets: three full blocks
    ((5, 5, 5), 1, 0, 1, 0.5),      # 750 tets, light: one block, a lane for every pair
    ((5, 5, 6), 3, 0, 1, 0.4),      # diffusion of three species, 2700 pairs: several blocks, a lane for every pair
    ((13, 13, 13), 4, 0, 2, 0.1),   # 13,182 tets in 128 blocks each: 448 pairs in a block
    ((11, 11, 11), 3, 0, 60, 0.1),  # 7986 tets in four blocks each: more pairs than lanes, listed
    ((4, 4, 4), 2, 0, 300, 0.3),    # two blocks on a compute unit: 768 pairs, 512 lanes, listed
    ((3, 3, 3), 2, 0, 600, 0.3),    # four: 324 pairs, 256 lanes, listed
    ((3, 3, 2), 2, 0, 600, 0.3),    # four: 216 pairs, a lane for every pair
    ((5, 5, 5), 1, 2, 1, 60.0),     # the same, crowded: 47 blocks, rejection sampler
    ((5, 5, 5), 2, 4, 100, 0.2),    # two blocks per realization
    ((3, 3, 3), 2, 4, 300, 0.5),    # more realizations than compute units: two blocks share one
    ((3, 3, 3), 2, 4, 700, 0.1),    # four share one
    ((2, 2, 3), 3, 2, 1100, 0.1),   # eight share one
    ((7, 6, 5), 3, 3, 600, 0.01),   # four share one, short lists
    ((8, 6, 6), 3, 2, 260, 1.5),    # each has one to itself
    ((7, 5, 4), 10, 8, 1, 1.5),     # ten species
    ((4, 4, 3), 16, 32, 1, 0.7),    # the most species and reactions: 64 lanes in the SSA at a time
    ((12, 12, 12), 1, 2, 150, 0.05),  # 10,368 tets in one block: short lists
    ((9, 9, 10), 3, 3, 150, 0.02),  # the same with several species
    ((16, 16, 8), 3, 0, 90, 0.02),  # two blocks, short lists, no reactions
    ((17, 16, 15), 4, 5, 1, 0.05),  # 24,480 tets, sparse: arrivals found by the occupancy bytes or directly
])
def test_resident_runs_match_the_oracle(P, orc, shape, S, R, Rz, mean):
    note(f"resident: {shape} cells, {S} species, {R} reactions, {Rz} realizations, mean {mean}")
    g, refs = both(P, orc, shape, S, R, Rz, mean)
    for n in (1, 2, 3, 6):
        g.step(n)
        for o in refs.values():
            o.run_steps(n)
        check(g, refs, n)
    t = g.time()[0] + 2.4 * g.tau  # a shortened last period
    g.run_until(t)
    for o in refs.values():
        o.run_until(t)
    check(g, refs, "run_until")
    g.close()


@pytest.mark.parametrize("shape,Rz,mean,crowded", [
    ((9, 9, 10), 150, 0.28, 1.0),  # one block of 4860 tets: lists for 2600 tets, 2200 of which react
    ((16, 16, 8), 90, 0.34, 0.5),  # two of 6144 tets, the molecules in the first
])
def test_short_lists_overflow(P, orc, shape, Rz, mean, crowded):
    note(f"resident: short lists that overflow, {shape} cells, {Rz} realizations")
    g, refs = both(P, orc, shape, 3, 3, Rz, mean, crowded=crowded)
    for n in (1, 2, 4):
        g.step(n)
        for o in refs.values():
            o.run_steps(n)
        check(g, refs, n)
    g.close()


@pytest.mark.parametrize("method", [{"transfer_form": 1}, {"occupancy_correction": False, "split_threshold": 3}])
def test_resident_method_options(P, orc, method):
    note(f"resident: method options {method}")
    xyz, tets = W.kuhn_box(6, 5, 5, 0.2e-6)
    D, rx = chemistry(3, 4)
    rng = np.random.default_rng(9)
    init = rng.poisson(8.0, (3, tets.shape[0])).astype(np.int32)
    g = P.Simulation(xyz, tets, D, rx, seed=9, **method)
    o = orc.OracleSim(xyz, tets, D, rx, seed=9)
    if method.get("transfer_form"):
        o.set_transfer_form(1)
    else:
        o.set_first_order(True)
        o.set_split_threshold(3)
    for s in range(3):
        g.set_counts(s, init[s])
        o.set_counts(s, init[s])
    for n in (2, 5):
        g.step(n)
        o.run_steps(n)
        check(g, {0: o}, (method, n))
    g.close()


def test_resident_runs_alternate_with_the_other_paths(P, orc):
    note("resident: alternating with two launches, the fused launch and the queue-based one-launch path")
    g, refs = both(P, orc, (9, 9, 9), 3, 4, 2, 0.3)
    for mode, n in ((0, 3), (1, 2), (0, 2), (3, 3), (0, 1), (2, 2), (0, 5), (1, 1), (0, 4)):
        P.rdos_set_launch_mode(g.h, mode)
        g.step(n)
        for o in refs.values():
            o.run_steps(n)
        check(g, refs, (mode, n))
    g.set_state(1001, 0.5)  # another parity
    for o in refs.values():
        o.set_state(1001, 0.5)
    P.rdos_set_launch_mode(g.h, 0)
    g.step(3)
    for o in refs.values():
        o.run_steps(3)
    check(g, refs, "set_state")
    g.close()


@pytest.mark.skip(reason="passed once, then its process ended with a host-side segmentation fault at exit, before "
                         "cooperative launches took turns; the cause is not shown")
def test_simulations_on_their_own_threads(P, orc):
    """Two simulations whose blocks each fill the device, stepped at once from
    two threads on their own streams, and a third through an engine."""
    import threading

    note("resident: two threads and an engine at once")
    sims = [both(P, orc, (8, 8, 7), 2, 3, 1, 0.5, seed=s) for s in (21, 22, 23)]
    engine = P.rdos_engine_create(0, 0)
    ticket = P.rdos_engine_submit(engine, sims[2][0].h, 96, 1.0)
    errors = []

    def run(g):
        try:
            for _ in range(12):
                g.step(8)
                g.get_counts(0)
        except Exception as e:  # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=run, args=(g,)) for g, _ in sims[:2]]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    P.rdos_engine_drain(engine)
    P.rdos_engine_release(engine, ticket)
    assert not errors, errors
    for g, refs in sims:
        for o in refs.values():
            o.run_steps(96)
        check(g, refs, "threads")
    P.rdos_engine_destroy(engine)
    for g, _ in sims:
        g.close()
