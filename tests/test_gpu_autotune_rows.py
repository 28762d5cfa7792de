"""The autotuner where workgroups evaluate the individuals: the launch shapes
stay as they are (no kernel reads them), and so do recorded generations; the
trajectory is the oracle's."""
import numpy as np
import pytest

from oracle import cnd_oracle as O
from paper_2412_20980_amd import inputs

pytestmark = pytest.mark.gpu


def test_single_ga():
    from paper_2412_20980_amd import gapa
    g = inputs.barabasi_albert(1000, 2, seed=3)
    graph = gapa.Graph.from_csr(g)
    other = dict(sweep_grid=777, band_scan=13, sweeps=1, band_blocks=99)
    graph.set_tuning(**other)
    ga, ref = gapa.GA(graph, 12, 40, 5, offspring=600, replay=True), O.OracleGA(g, 12, 40, 5, offspring=600)
    ga.step(1)
    ga.record(3)
    assert ga.autotune(reps=1) == other and graph.get_tuning() == other
    ga.record(3)  # (refused after a change of shapes, until a generation has run)
    ga.step(3)
    for _ in range(4):
        ref.step()
    rows, F = ga.population()
    assert np.array_equal(rows, ref.pop) and np.array_equal(F, ref.F)


def test_batch():
    from paper_2412_20980_amd import gapa
    gs = [inputs.barabasi_albert(n, 2, seed=n) for n in (300, 900)]
    params = [dict(k=8, pop=20, seed=b) for b in range(2)]
    bt = gapa.Batch([gapa.Graph.from_csr(g) for g in gs], params, replay=True)
    bt.step(1)
    bt.record(2)
    before = bt.get_tuning()
    assert bt.autotune(reps=1) == before == bt.get_tuning()
    bt.record(2)
    bt.step(2)
    for b, g in enumerate(gs):
        ref = O.OracleGA(g, 8, 20, b)
        for _ in range(3):
            ref.step()
        rows, F = bt.population(b)
        assert np.array_equal(rows, ref.pop) and np.array_equal(F, ref.F)
