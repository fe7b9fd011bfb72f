"""Repeated reads of one simulation: the pinned read-out of small rows (from a
simulation's fifth read on, up to 64 KB with the flags word) against the
zero-copy view, and again after every simulation has gone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("box", [(1, 1, 1), (13, 14, 15), (14, 14, 14)])  # 6, 16380 and 16464 tets
def test_repeated_reads_equal_the_view(box):
    import paper_1512_03126_amd as P
    import workloads as W

    for _ in range(2):
        xyz, tets = W.kuhn_box(*box, 0.1e-6)
        T = tets.shape[0]
        sim = P.Simulation(xyz, tets, [1e-12, 2e-12], [], seed=7)
        start = [np.random.default_rng(s).poisson(2.0, T).astype(np.int32) for s in range(2)]
        for s in range(2):
            sim.set_counts(s, start[s])
        for s in range(2):
            np.testing.assert_array_equal(sim.get_counts(s), start[s])
        for _ in range(4):
            sim.step(1)
            for s in range(2):
                got = sim.get_counts(s)
                np.testing.assert_array_equal(got, sim.device_counts(s, 0).cpu().numpy()[:T])
                assert got.sum() == start[s].sum()
        sim.close()
