"""The scratch that sparse batches run with stays within the engine's memory
budget, and an admission gets it back."""
import sys
import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

Rz, N, MOLECULES = 300, 20, 2600  # 48,000 tets: 16,384 slots of 36 bytes a realization, 177 MB of scratch


def note(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


def batch(P, orc, seed):
    xyz, tets = W.kuhn_lattice(N, 0.1e-6)
    T = tets.shape[0]
    D, rx = [1e-12, 2e-12, 0.5e-12], [([0, 1], [2], 1e8), ([2], [0, 1], 300.0)]
    rng = np.random.default_rng(seed)
    init = np.stack([np.bincount(rng.integers(0, T, MOLECULES), minlength=T) for _ in range(3)]).astype(np.int32)
    g = P.Simulation(xyz, tets, D, rx, seed=seed, n_realizations=Rz)
    o = orc.OracleSim(xyz, tets, D, rx, seed=seed, realization=Rz - 1)
    for s in range(3):
        for r in range(Rz):
            g.set_counts(s, init[s], realization=r)
        o.set_counts(s, init[s])
    return g, o


def check(P, e, ticket, g, o, n):
    P.rdos_engine_release(e, ticket)
    o.run_steps(n)
    assert np.array_equal(g.get_counts(None, realization=Rz - 1), o.get_counts())


def test_scratch_stays_within_the_budget(P_orc):
    P, orc = P_orc
    import torch

    note("budget: a sparse batch whose scratch fits, one whose scratch does not, and an admission that takes it back")
    (a, oa), (b, ob) = batch(P, orc, 5), batch(P, orc, 6)
    need = a.info()["device_bytes"]

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    def scratch_of(e):
        before = free()
        P.rdos_engine_destroy(e)
        return free() - before

    e = P.rdos_engine_create(0, 0)  # tunes the queue for this size, then runs in LDS
    t = P.rdos_engine_submit(e, a.h, 340, 1.0)
    P.rdos_engine_drain(e)
    check(P, e, t, a, oa, 340)
    assert scratch_of(e) > 150e6

    e = P.rdos_engine_create(0, int(need + 100e6))  # no room for the scratch: the queue runs the periods
    t = P.rdos_engine_submit(e, a.h, 20, 1.0)
    P.rdos_engine_drain(e)
    check(P, e, t, a, oa, 20)
    assert scratch_of(e) < 50e6

    e = P.rdos_engine_create(0, int(2 * need + 50e6))  # room until the second batch comes
    before = free()
    t = P.rdos_engine_submit(e, a.h, 1500, 1.0)
    time.sleep(0.02)
    assert before - free() > 150e6
    t2 = P.rdos_engine_submit(e, b.h, 40, 1.0)
    P.rdos_engine_drain(e)
    check(P, e, t, a, oa, 1500)
    check(P, e, t2, b, ob, 40)
    P.rdos_engine_destroy(e)
    a.close()
    b.close()


@pytest.fixture
def P_orc(orc):
    import paper_1512_03126_amd as P

    P.lib()
    return P, orc
