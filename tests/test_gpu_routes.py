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


def least_times(P, g, n, calls):
    least = {0: np.inf, 1: np.inf}
    for i in range(calls + 3):
        for mode in least:
            P.rdos_set_launch_mode(g.h, mode)
            t = time.perf_counter()
            g.step(n)
            g.synchronize()
            if i >= 3:
                least[mode] = min(least[mode], time.perf_counter() - t)
    P.rdos_set_launch_mode(g.h, 0)
    return least


def box(P, shape, S, mean, Rz=1):
    xyz, tets = W.kuhn_box(*shape, 0.1e-6)
    T = tets.shape[0]
    rng = np.random.default_rng(6)
    g = P.Simulation(xyz, tets, [1e-12] * S, [], seed=6, n_realizations=Rz)
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
    least = least_times(P, g, n, 40)
    assert least[0] <= 1.12 * least[1], least
    g.close()
