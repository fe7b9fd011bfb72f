"""The path that a call takes by itself is no slower than two launches per
period, where a rule on its length or on what the tets hold decides (both
timed in turn, the least of many calls)."""
import sys
import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def note(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


def least_times(P, g, n, calls, limit):
    """The least times of launch modes 0 and 1, by more calls (up to three
    times as many) while their ratio is above the limit; and the periods run."""
    least, steps = {0: np.inf, 1: np.inf}, 0
    for i in range(3 * calls + 3):
        for mode in least:
            P.rdos_set_launch_mode(g.h, mode)
            t = time.perf_counter()
            g.step(n)
            g.synchronize()
            steps += n
            if i >= 3:
                least[mode] = min(least[mode], time.perf_counter() - t)
        if i >= 3 and (i - 2) % calls == 0 and least[0] <= limit * least[1]:
            break
    P.rdos_set_launch_mode(g.h, 0)
    return least, steps


def box(P, shape, S, mean, Rz=1, rx=()):
    xyz, tets = W.kuhn_box(*shape, 0.1e-6)
    T = tets.shape[0]
    rng = np.random.default_rng(6)
    g = P.Simulation(xyz, tets, [1e-12] * S, rx, seed=6, n_realizations=Rz)
    init = rng.poisson(mean, (Rz, S, T)).astype(np.int32)
    for r in range(Rz):
        for s in range(S):
            g.set_counts(s, init[r, s], realization=r)
    return g, (xyz, tets, init)


@pytest.mark.parametrize("shape,S,Rz,mean,n", [
    ((70, 70, 70), 1, 1, 0.01, 2),  # most counts are empty: reading them all costs more than two periods save
    ((70, 70, 70), 1, 1, 0.01, 3),
    ((3, 3, 3), 2, 3000, 0.01, 1),  # a block per realization
])
def test_short_runs_of_sparse_lists(shape, S, Rz, mean, n):
    import paper_1512_03126_amd as P

    note(f"routes: {n} periods a call, {shape} cells, {S} species, {Rz} realizations at {mean}")
    g, _ = box(P, shape, S, mean, Rz)
    least, _ = least_times(P, g, n, 40, 1.12)
    print("least", least, flush=True)
    assert least[0] <= 1.12 * least[1], least
    g.close()


@pytest.mark.parametrize("shape,S,Rz,mean,n", [
    ((20, 20, 20), 3, 10, 0.01, 3),
    ((55, 55, 55), 4, 1, 0.001, 4),
])
def test_short_requests_of_sparse_lists(orc, shape, S, Rz, mean, n):
    import paper_1512_03126_amd as P

    note(f"routes: requests of {n} periods, {shape} cells, {S} species, {Rz} realizations at {mean}")
    g, (xyz, tets, init) = box(P, shape, S, mean, Rz)
    engines = [P.rdos_engine_create(0, 0) for _ in range(2)]
    P.rdos_engine_set_shape(engines[1], 32, 2048, 1, 1)  # a fixed shape runs over the queue
    least = [np.inf, np.inf]
    steps = 0
    for i in range(63):
        for j, e in enumerate(engines):
            t = time.perf_counter()
            ticket = P.rdos_engine_submit(e, g.h, n, 1.0)
            P.rdos_engine_drain(e)
            P.rdos_engine_release(e, ticket)
            steps += n
            if i >= 3:
                least[j] = min(least[j], time.perf_counter() - t)
        if i >= 22 and least[0] <= 1.12 * least[1]:
            break
    for e in engines:
        P.rdos_engine_destroy(e)
    print("least", least, flush=True)
    assert least[0] <= 1.12 * least[1], least
    o = orc.OracleSim(xyz, tets, [1e-12] * S, [], seed=6, realization=Rz - 1)
    for s in range(S):
        o.set_counts(s, init[Rz - 1, s])
    o.run_steps(steps)
    assert np.array_equal(g.get_counts(None, realization=Rz - 1), o.get_counts())
    g.close()


def chain(S, R):
    """R reactions over S species that keep the number of molecules."""
    rx = []
    for q in range(R):
        a, b, c = q % S, (q + 1) % S, (q + 2) % S
        rx.append([([a, b], [c, a], 2e8), ([a], [b], 60.0), ([a, a], [b, c], 1e8), ([b], [c], 90.0)][q % 4])
    return rx


@pytest.mark.parametrize("shape,S,R,Rz,mean", [
    ((4, 4, 4), 16, 32, 1000, 0.3),  # 64 lanes of a compute unit in the SSA, in four turns
    ((5, 5, 5), 10, 24, 200, 0.3),   # as few in a block of 750 tets
    ((2, 2, 2), 3, 2, 12000, 0.01),  # many turns with nearly nothing to do
])
def test_models_that_leave_lds_behind(orc, shape, S, R, Rz, mean):
    import paper_1512_03126_amd as P

    note(f"routes: {Rz} realizations, {shape} cells, {S} species, {R} reactions at {mean}")
    xyz, tets = W.kuhn_box(*shape, 0.2e-6)
    T = tets.shape[0]
    rng = np.random.default_rng(8)
    D = [1e-12 * (0.3 + 0.1 * s) for s in range(S)]
    g = P.Simulation(xyz, tets, D, chain(S, R), seed=8, n_realizations=Rz)
    o = orc.OracleSim(xyz, tets, D, chain(S, R), seed=8, realization=Rz - 1)
    init = rng.poisson(mean, (S, T)).astype(np.int32)
    for s in range(S):
        for r in range(Rz):
            g.set_counts(s, init[s], realization=r)
        o.set_counts(s, init[s])
    least, steps = least_times(P, g, 10, 12, 1.12)
    print("least", least, flush=True)
    assert least[0] <= 1.12 * least[1], least
    o.run_steps(steps)
    assert np.array_equal(g.get_counts(None, realization=Rz - 1), o.get_counts())
    g.close()


def test_crowded_views_leave_the_short_lists():
    """Counts that a device view made crowded, after they were set sparse: the
    first run finds its lists too short, later ones go over the queue until
    counts are set again."""
    import torch

    import paper_1512_03126_amd as P

    note("routes: 998,250 tets of four species set at 0.01 and written through a view at 1 molecule per pair")
    g, (_, tets, init) = box(P, (55, 55, 55), 4, 0.01, rx=[([0, 1], [2], 2e8), ([2], [0, 1], 400.0)])
    crowd = torch.from_numpy(np.random.default_rng(3).poisson(1.0, tets.shape[0]).astype(np.int32))
    for s in range(4):
        g.device_counts(s, 0).copy_(crowd)
    torch.cuda.synchronize()
    g.step(8)
    g.synchronize()
    least, _ = least_times(P, g, 8, 12, 1.1)
    print("least", least, flush=True)
    assert least[0] <= 1.1 * least[1], least
    for s in range(4):
        g.set_counts(s, init[0, s])
    least, _ = least_times(P, g, 8, 12, 0.9)
    print("least", least, flush=True)
    assert least[0] <= 0.9 * least[1], least  # LDS again
    g.close()


def test_crowded_views_in_the_engine(orc):
    """The same through an engine, with a look at every count: a run whose
    lists overflow, one over the queue, and one in LDS after counts are set."""
    import torch

    import paper_1512_03126_amd as P

    Rz = 150
    note(f"routes: {Rz} realizations of 4860 tets written crowded through views, engine and plain")
    xyz, tets = W.kuhn_box(9, 9, 10, 0.2e-6)
    T = tets.shape[0]
    rx = [([0, 1], [2], 2e8), ([2], [0, 1], 60.0)]
    D = [1e-12, 0.5e-12, 0.8e-12]
    rng = np.random.default_rng(4)
    g = P.Simulation(xyz, tets, D, rx, seed=9, n_realizations=Rz, tau_scale=None)
    e = P.rdos_engine_create(0, 0)
    sparse = (rng.random((3, T)) < 0.01).astype(np.int32)
    crowd = rng.poisson(0.5, (3, T)).astype(np.int32)
    o = orc.OracleSim(xyz, tets, D, rx, seed=9, realization=Rz - 1)

    def request(n):
        t = P.rdos_engine_submit(e, g.h, n, 1.0)
        P.rdos_engine_drain(e)
        P.rdos_engine_release(e, t)
        o.run_steps(n)
        assert np.array_equal(g.get_counts(None, realization=Rz - 1), o.get_counts()), n

    def sets(counts, view):
        for r in range(Rz):
            for s in range(3):
                if view:
                    g.device_counts(s, r).copy_(torch.from_numpy(counts[s]))
                else:
                    g.set_counts(s, counts[s], realization=r)
        torch.cuda.synchronize()
        for s in range(3):
            o.set_counts(s, counts[s])

    sets(sparse, False)
    request(9)
    sets(crowd, True)
    request(11)
    request(12)
    g.step(5)
    o.run_steps(5)
    sets(sparse, False)
    sets(crowd, True)
    for n in (3, 4, 2):  # in LDS, and not looked at between
        g.step(n)
        o.run_steps(n)
    assert np.array_equal(g.get_counts(None, realization=Rz - 1), o.get_counts())
    sets(sparse, False)
    request(10)
    g.step(6)
    o.run_steps(6)
    assert np.array_equal(g.get_counts(None, realization=Rz - 1), o.get_counts())
    P.rdos_engine_destroy(e)
    g.close()


def test_reacting_batches_leave_the_sparse_kernel(orc):
    """A batch whose molecules react within a few periods: the estimate takes
    the sparse kernel, a trial finds the queue faster."""
    import paper_1512_03126_amd as P

    Rz, S = 300, 3
    note(f"routes: {Rz} realizations of 14,196 tets, three species that react within a few periods")
    xyz, tets = W.kuhn_box(13, 13, 14, 0.2e-6)
    T = tets.shape[0]
    D, rx = [0.3e-12, 0.4e-12, 0.5e-12], [([0], [1], 300.0), ([1], [0], 200.0), ([0, 2], [1], 1e8)]
    g = P.Simulation(xyz, tets, D, rx, seed=12, n_realizations=Rz)
    engines = [P.rdos_engine_create(0, 0) for _ in range(2)]
    P.rdos_engine_set_shape(engines[1], 32, 2048, 2, 1)

    def request(e, n):
        t = time.perf_counter()
        ticket = P.rdos_engine_submit(e, g.h, n, 1.0)
        P.rdos_engine_drain(e)
        P.rdos_engine_release(e, ticket)
        return time.perf_counter() - t

    request(engines[0], 331)  # empty: the queue is tuned for lists of this size
    rng = np.random.default_rng(12)
    init = np.stack([np.bincount(rng.integers(0, T, 1000), minlength=T) for _ in range(S)]).astype(np.int32)
    for s in range(S):
        for r in range(Rz):
            g.set_counts(s, init[s], realization=r)
    o = orc.OracleSim(xyz, tets, D, rx, seed=12, realization=Rz - 1)
    for s in range(S):
        o.set_counts(s, init[s])
    t, k = g.time()
    o.set_state(k, t)
    request(engines[0], 80)
    least = [np.inf, np.inf]
    steps = 80
    for i in range(24):
        for j, e in enumerate(engines):
            least[j] = min(least[j], request(e, 32))
            steps += 32
        if i >= 7 and least[0] <= 1.15 * least[1]:
            break
    for e in engines:
        P.rdos_engine_destroy(e)
    o.run_steps(steps)
    assert np.array_equal(g.get_counts(None, realization=Rz - 1), o.get_counts())
    g.close()
    print("least", least, flush=True)
    assert least[0] <= 1.15 * least[1], least


def test_geometry_of_small_meshes_by_one_copy(orc):
    """On both sides of the size from which the device takes the tables apart
    (16,384 tets), against the oracle's; a small mesh's cost no more than a few
    waits."""
    import paper_1512_03126_amd as P

    for shape in ((5, 5, 5), (13, 14, 15), (14, 14, 14)):
        xyz, tets = W.kuhn_box(*shape, 0.2e-6)
        note(f"routes: geometry of {tets.shape[0]} tets")
        g = P.Simulation(xyz, tets, [1e-12], [], seed=1)
        o = orc.OracleSim(xyz, tets, [1e-12], [], seed=1)
        got, want = g.geometry(), o.geometry()
        assert np.array_equal(got["nbr"], want["nbr"])
        for k in ("w", "g", "nav"):
            np.testing.assert_allclose(got[k], want[k], rtol=1e-13)
        if tets.shape[0] == 750:
            def least(call):
                times = []
                for _ in range(40):
                    t = time.perf_counter()
                    call()
                    times.append(time.perf_counter() - t)
                return min(times)
            assert least(g.geometry) <= 2.5 * least(g.synchronize)
        g.close()
