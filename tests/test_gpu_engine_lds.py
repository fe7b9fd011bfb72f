"""Work lists that the engine runs with their state in LDS, against the
oracle: mixes of requests cut into blocks (several sizes, species counts and
lengths, requests that join and leave), and batches of sparse realizations,
one block each, with a hash table of their occupied pairs; a batch whose
table overflows falls back to the queue with nothing lost."""
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


RX = [([0, 1], [2], 3e8), ([2], [0, 1], 400.0), ([0, 0], [1], 1e8)]


def request(P, orc, n, S, Rz, mean, seed, rx=RX, **method):
    xyz, tets = W.tiny_lattice(n, 0.2e-6, jitter_frac=0.2, seed=seed)
    T = tets.shape[0]
    D = [1e-12 * (0.4 + 0.3 * s) for s in range(S)]
    rng = np.random.default_rng(seed)
    init = rng.poisson(mean, (Rz, S, T)).astype(np.int32)
    g = P.Simulation(xyz, tets, D, rx, seed=seed, n_realizations=Rz, tau_scale=None, **method)
    refs = {}
    for r in range(Rz):
        for s in range(S):
            g.set_counts(s, init[r, s], realization=r)
    for r in sorted({0, Rz - 1}):
        o = orc.OracleSim(xyz, tets, D, rx, seed=seed, realization=r)
        if method.get("transfer_form"):
            o.set_transfer_form(1)
        for s in range(S):
            o.set_counts(s, init[r, s])
        refs[r] = o
    return g, refs


def finish(P, e, ticket, g, refs, n, what):
    P.rdos_engine_release(e, ticket)
    for r, o in refs.items():
        o.run_steps(n)
        got, want = g.get_counts(None, realization=r), o.get_counts()
        assert np.array_equal(got, want), (what, r, int((got != want).sum()))


def test_mixed_requests_in_blocks(P, orc):
    note("engine: a mix of requests with their counts in LDS")
    e = P.rdos_engine_create(0, 0)
    specs = [(2, 3, 1, 2.0, 71), (9, 3, 2, 0.1, 70), (6, 5, 1, 1.5, 33), (5, 16, 1, 0.4, 41), (12, 3, 1, 0.02, 97)]
    sims = [request(P, orc, n, S, Rz, mean, 40 + i) for i, (n, S, Rz, mean, _) in enumerate(specs)]
    sims.append(request(P, orc, 4, 3, 1, 6.0, 60, transfer_form=1))
    steps = [x[4] for x in specs] + [50]
    tickets = [P.rdos_engine_submit(e, g.h, k, 1.0) for (g, _), k in zip(sims, steps)]
    P.rdos_engine_drain(e)
    for i, ((g, refs), t, k) in enumerate(zip(sims, tickets, steps)):
        finish(P, e, t, g, refs, k, f"request {i}")
    # a second run of two of them, continuing
    tickets = [P.rdos_engine_submit(e, sims[i][0].h, 5, 1.0) for i in (1, 4)]
    P.rdos_engine_drain(e)
    for i, t in zip((1, 4), tickets):
        finish(P, e, t, *sims[i], 5, f"request {i} again")
    P.rdos_engine_destroy(e)
    for g, _ in sims:
        g.close()


def test_many_small_realizations_take_turns(P, orc):
    note("engine: more realizations than compute units, one block each")
    e = P.rdos_engine_create(0, 0)
    sims = [request(P, orc, 3, 3, 300, 0.5, 7), request(P, orc, 2, 3, 90, 2.0, 8)]
    P.rdos_engine_hold(e, True)
    tickets = [P.rdos_engine_submit(e, g.h, k, 1.0) for (g, _), k in zip(sims, (45, 30))]
    P.rdos_engine_hold(e, False)
    P.rdos_engine_drain(e)
    for (g, refs), t, k in zip(sims, tickets, (45, 30)):
        finish(P, e, t, g, refs, k, "small")
    P.rdos_engine_destroy(e)
    for g, _ in sims:
        g.close()


def batch(P, orc, n, Rz, seed, form=0):
    """A+B<->C on n^3 cells of 0.1 um at the batch's concentration."""
    m = W.abc_lattice(n=n, a=0.1e-6, seed=seed, n_realizations=Rz)
    rx = [([0, 1], [2], 1e8), ([2], [0, 1], 300.0)]  # reactions in most periods
    g = P.Simulation(m.xyz, m.tets, m.D, rx, seed=seed, n_realizations=Rz, transfer_form=form)
    refs = {}
    for r in range(Rz):
        for s in range(3):
            g.set_counts(s, m.init[r, s], realization=r)
    for r in (0, Rz - 1):
        o = orc.OracleSim(m.xyz, m.tets, m.D, rx, seed=seed, realization=r)
        if form:
            o.set_transfer_form(1)
        for s in range(3):
            o.set_counts(s, m.init[r, s])
        refs[r] = o
    return g, refs


@pytest.mark.parametrize("form", [0, 1])
def test_sparse_batch_matches_the_oracle(P, orc, form):
    note(f"engine: sparse batch, transfer form {form}")
    e = P.rdos_engine_create(0, 0)
    sims = [batch(P, orc, 18, 40, 3, form), batch(P, orc, 13, 9, 4, form)]
    for n in (331, 32, 7, 1):  # the tuner's periods over the queue come first
        P.rdos_engine_hold(e, True)
        tickets = [P.rdos_engine_submit(e, g.h, n, 1.0) for g, _ in sims]
        P.rdos_engine_hold(e, False)
        P.rdos_engine_drain(e)
        for (g, refs), t in zip(sims, tickets):
            finish(P, e, t, g, refs, n, (form, n))
    # and back over the plain path
    for g, refs in sims:
        g.step(3)
        for r, o in refs.items():
            o.run_steps(3)
            assert np.array_equal(g.get_counts(None, realization=r), o.get_counts())
    P.rdos_engine_destroy(e)
    for g, _ in sims:
        g.close()


def test_full_table_falls_back_to_the_queue(P, orc):
    note("engine: a sparse batch with one crowded realization (written through the device view)")
    import torch

    n, Rz, crowded = 20, 64, 17
    xyz, tets = W.kuhn_lattice(n, 0.1e-6)
    T = tets.shape[0]
    D, rx = [1e-12, 2e-12], [([0, 1], [0], 1e8)]
    rng = np.random.default_rng(2)
    init = np.zeros((Rz, 2, T), np.int32)
    for r in range(Rz):
        for s in range(2):
            np.add.at(init[r, s], rng.integers(0, T, 300), 1)
    g = P.Simulation(xyz, tets, D, rx, seed=3, n_realizations=Rz)
    for r in range(Rz):
        for s in range(2):
            g.set_counts(s, init[r, s], realization=r)
    init[crowded] = rng.poisson(0.7, (2, T)).astype(np.int32)  # about 48,000 pairs
    for s in range(2):
        g.device_counts(s, crowded).copy_(torch.from_numpy(init[crowded, s]))
    torch.cuda.synchronize()
    e = P.rdos_engine_create(0, 0)
    t = P.rdos_engine_submit(e, g.h, 340, 1.0)
    P.rdos_engine_drain(e)
    P.rdos_engine_release(e, t)
    for r in (0, crowded):
        o = orc.OracleSim(xyz, tets, D, rx, seed=3, realization=r)
        for s in range(2):
            o.set_counts(s, init[r, s])
        o.run_steps(340)
        got, want = g.get_counts(None, realization=r), o.get_counts()
        assert np.array_equal(got, want), (r, int((got != want).sum()))
    P.rdos_engine_destroy(e)
    g.close()
