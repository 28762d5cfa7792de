"""Further pull rounds with few blocks, and left out: lattices and random graphs
too deep or too large for workgroups, at one word a node (no rounds on the
lattices) and more, a graph in pieces (none), a batch whose union has rounds
though its parts are small; against the oracle."""
import numpy as np
import pytest

from oracle import cnd_oracle as O
from paper_2412_20980_amd import inputs

pytestmark = pytest.mark.gpu


def lattice(a, b):
    i = np.random.default_rng(a).permutation(a * b).reshape(a, b)
    return inputs.csr_from_edges(a * b, np.concatenate([i[:, :-1].ravel(), i[:-1].ravel()]),
                                 np.concatenate([i[:, 1:].ravel(), i[1:].ravel()]))


def pairs(n):
    i = np.arange(0, n, 2)
    return inputs.csr_from_edges(n, i, i + 1)


@pytest.mark.parametrize("name,make", [("lattice", lambda: lattice(135, 140)), ("larger lattice", lambda: lattice(260, 261)),
                                       ("random", lambda: inputs.erdos_renyi(65_600, 5.0, seed=2)),
                                       ("pairs", lambda: pairs(50_000))])
@pytest.mark.parametrize("P", [1, 32, 33, 100])
def test_matches_oracle(name, make, P):
    from paper_2412_20980_amd import gapa
    g = make()
    rows = inputs.random_population(g.n, g.n // 40, P, seed=P)
    print(f"{name} n={g.n} P={P}", flush=True)
    F, M = gapa.Graph.from_csr(g).eval(rows, want_mcn=True)
    Fo, Mo = O.eval_population(g, rows, want_mcn=True)
    assert np.array_equal(F, Fo) and np.array_equal(M, Mo)


def test_batch_with_a_deep_graph():
    from paper_2412_20980_amd import gapa
    gs = [lattice(135, 140), lattice(3, 5), inputs.erdos_renyi(400, 3.0, seed=1)]
    params = [dict(k=max(1, g.n // 30), pop=9, seed=b) for b, g in enumerate(gs)]
    bt = gapa.Batch([gapa.Graph.from_csr(g) for g in gs], params)
    bt.step(2)
    for b, g in enumerate(gs):
        ref = O.OracleGA(g, params[b]["k"], 9, b)
        ref.step()
        ref.step()
        rows, F = bt.population(b)
        assert np.array_equal(rows, ref.pop) and np.array_equal(F, ref.F)
