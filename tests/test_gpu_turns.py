"""Several simulations whose blocks wait for each other in one process: on
streams that come and go, beside a stream that its owner captures, and while
another's run is under way.  Every count against the oracle."""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

D = [1e-12, 0.5e-12, 0.8e-12]
RX = [([0, 1], [2], 2e8), ([2], [0, 1], 400.0)]


def note(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    import paper_1512_03126_amd as mod

    mod.lib()
    return mod


def pair(P, orc, cells, seed):
    """A reacting box of several blocks (1080 tet-species and more) and its
    oracle."""
    xyz, tets = W.kuhn_box(*cells, 0.2e-6)
    init = np.random.default_rng(seed).poisson(3.0, (3, tets.shape[0])).astype(np.int32)
    g = P.Simulation(xyz, tets, D, RX, seed=seed)
    o = orc.OracleSim(xyz, tets, D, RX, seed=seed)
    for s in range(3):
        g.set_counts(s, init[s])
        o.set_counts(s, init[s])
    return g, o


def check(g, o, what):
    got, want = g.get_counts(), o.get_counts()
    assert np.array_equal(got, want), (what, int((got != want).sum()))


def through_engine(P, e, g, n):
    t = P.rdos_engine_submit(e, g.h, n, 1.0)
    P.rdos_engine_drain(e)
    P.rdos_engine_release(e, t)


def test_streams_come_and_go(P, orc):
    note("turns: simulations and engines one after the other, each on a stream of its own")
    import torch

    for i in range(6):
        g, o = pair(P, orc, (4, 4, 4 + i % 2), 10 + i)
        g.step(5)
        o.run_steps(5)
        if i % 3 == 1:  # its launches go on on another stream
            st = torch.cuda.Stream()
            g.set_stream(st.cuda_stream)
            g.step(4)
            o.run_steps(4)
            g.set_stream(None)
            del st
        e = P.rdos_engine_create(0, 0)
        through_engine(P, e, g, 40)
        o.run_steps(40)
        g.step(3)
        o.run_steps(3)
        P.rdos_engine_destroy(e)
        check(g, o, i)
        g.close()


def test_one_stream_for_two(P, orc):
    note("turns: two simulations stepped in turn on one stream of the caller's")
    import torch

    st = torch.cuda.Stream()
    sims = [pair(P, orc, (4, 4, 5), 30 + i) for i in range(2)]
    for g, _ in sims:
        g.set_stream(st.cuda_stream)
    for n in (3, 1, 6):
        for g, o in sims:
            g.step(n)
            o.run_steps(n)
    for i, (g, o) in enumerate(sims):
        check(g, o, i)
        g.close()


def test_beside_a_captured_stream(P, orc):
    note("turns: a run while the stream of the last one is captured by its owner")
    import torch

    st = torch.cuda.Stream()
    (a, oa), (b, ob) = pair(P, orc, (4, 4, 5), 40), pair(P, orc, (4, 4, 4), 41)
    a.set_stream(st.cuda_stream)
    a.step(5)
    P.rdos_step_static(a.h, 1)
    oa.run_steps(6)
    check(a, oa, "before")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(st):
        graph.capture_begin(capture_error_mode="thread_local")
        P.rdos_step_static(a.h, 2)
        b.step(4)
        graph.capture_end()
    ob.run_steps(4)
    check(b, ob, "beside the capture")
    with torch.cuda.stream(st):
        graph.replay()
    st.synchronize()
    oa.run_steps(2)
    check(a, oa, "replayed")
    a.step(3)
    oa.run_steps(3)
    check(a, oa, "after")
    a.close()
    b.close()


def test_beside_a_run_under_way(P, orc):
    note("turns: short runs, one to a shortened last period and one through an engine, beside a long one")
    (a, oa), (b, ob), (c, oc) = (pair(P, orc, cells, 50 + i) for i, cells in enumerate([(2, 2, 4), (4, 4, 4), (4, 5, 4)]))
    e = P.rdos_engine_create(0, 0)
    a.step(20000)  # about a tenth of a second
    b.step(70)
    t_end = b.time()[0] + 90.4 * b.tau
    b.run_until(t_end)
    through_engine(P, e, c, 100)
    b.step(5)
    oa.run_steps(20000)
    ob.run_steps(70)
    ob.run_until(t_end)
    ob.run_steps(5)
    oc.run_steps(100)
    check(b, ob, "beside")
    check(c, oc, "engine")
    check(a, oa, "the long run")
    P.rdos_engine_destroy(e)
    for g in (a, b, c):
        g.close()


@pytest.mark.parametrize("modes", [(0, 2), (2, 0), (2, 2)])
def test_one_launch_over_the_queue_takes_its_turn(P, orc, modes):
    note(f"turns: launch mode {modes[1]} beside a long run in launch mode {modes[0]}")
    (a, oa), (b, ob) = pair(P, orc, (2, 2, 4), 60), pair(P, orc, (4, 4, 4), 61)
    P.rdos_set_launch_mode(a.h, modes[0])
    P.rdos_set_launch_mode(b.h, modes[1])
    a.step(7000)  # two launches
    t_end = b.time()[0] + 60.4 * b.tau
    b.run_until(t_end)
    ob.run_until(t_end)
    check(b, ob, "beside")
    a.synchronize()
    for n in (3, 2):  # and in turn again
        b.step(n)
        ob.run_steps(n)
    check(b, ob, "after")
    oa.run_steps(7000)
    check(a, oa, "the long run")
    a.close()
    b.close()


def test_runs_wait_on_the_device(P, orc):
    note("turns: three simulations stepped in turn without a wait, one of them with a long run between")
    sims = [pair(P, orc, cells, 70 + i) for i, cells in enumerate([(4, 4, 4), (4, 4, 5), (2, 2, 4)])]
    for n in (40, 1, 25, 60):
        for i, (g, o) in enumerate(sims):
            k = 900 if n == 25 and i == 1 else n  # the others' next runs are too short to wait for it
            g.step(k)
            o.run_steps(k)
    g, o = pair(P, orc, (4, 4, 4), 80)  # a simulation closed while the others' runs are under way
    g.step(30)
    o.run_steps(30)
    check(g, o, "closed")
    g.close()
    for i, (g, o) in enumerate(sims):
        t_end = g.time()[0] + 20.4 * g.tau
        g.run_until(t_end)
        o.run_until(t_end)
    for i, (g, o) in enumerate(sims):
        check(g, o, i)
        g.close()
