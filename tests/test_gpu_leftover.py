"""Sweeps over all nodes where the list of open nodes outgrows LDS: nodes that
are components of their own (a star without its centre, few or all of its
leaves), small pieces, a list that fits after such a sweep and one that never
does, for one individual a block, a few and eight; every row against the
library's edge-parallel union-find, a sample against the oracle."""
import numpy as np
import pytest

from oracle import cnd_oracle as O
from paper_2412_20980_amd import inputs

pytestmark = pytest.mark.gpu


def pieces(n, size, star):
    """Stars or paths of `size` nodes, a random graph of 3000 nodes beside them."""
    core = inputs.erdos_renyi(3000, 6.0, seed=2)
    i = np.arange(3000, n)
    at = (i - 3000) % size
    u, v = (i - at, i) if star else (i - 1, i)
    src = np.repeat(np.arange(3000), np.diff(core.row_ptr))
    p = np.random.default_rng(n).permutation(n)
    return inputs.csr_from_edges(n, p[np.concatenate([src, u[at != 0]])], p[np.concatenate([core.col_idx, v[at != 0]])])


@pytest.mark.parametrize("n,size,star", [(65_000, 62_000, True), (60_000, 100, True), (50_000, 2, True),
                                         (40_000, 30, False), (24_500, 24_500, True)])
@pytest.mark.parametrize("P", [130, 700, 2060])
def test_matches_union_find_and_oracle(n, size, star, P):
    from paper_2412_20980_amd import gapa
    g = pieces(n, size, star)
    rng = np.random.default_rng(P)
    k = 700
    top = np.argsort(-g.degrees(), kind="stable")[:k]
    rows = np.concatenate([np.tile(top[:k // 2], (P, 1)), rng.integers(0, n, size=(P, k // 2))], axis=1)
    rows[1::3, :k // 2] = rng.integers(0, n, size=(len(rows[1::3]), k // 2))  # hubs stay
    rows = rows.astype(np.int32)
    print(f"n={n} size={size} star={star} P={P}", flush=True)
    F, M = gapa.Graph.from_csr(g).eval(rows, want_mcn=True)
    Fu, Mu = gapa.Graph.from_csr(g, unionfind=True).eval(rows, want_mcn=True)
    assert np.array_equal(F, Fu) and np.array_equal(M, Mu)
    idx = [0, 1, P - 1]
    Fo, Mo = O.eval_population(g, rows[idx], want_mcn=True)
    assert np.array_equal(F[idx], Fo) and np.array_equal(M[idx], Mo)


@pytest.mark.parametrize("n,edges", [(63, 0), (64, 3), (65, 0), (20_001, 150)])
def test_isolated_survivors_decide_mcn(n, edges):
    """Every node with an edge removed, and of the isolated ones all but the last,
    the first, one or none, for as many individuals as a block takes."""
    from paper_2412_20980_amd import gapa
    g = inputs.csr_from_edges(n, np.arange(edges), np.arange(edges) + edges)
    order = np.argsort(-g.degrees(), kind="stable").astype(np.int32)
    keep = [n - 1, 2 * edges, (n + 2 * edges) // 2, None]
    rows = np.stack([order if z is None else np.where(order == order[z], order[(z + 1) % n], order) for z in keep])
    rows = np.tile(rows, (513, 1))
    F, M = gapa.Graph.from_csr(g).eval(rows, want_mcn=True)
    Fo, Mo = O.eval_population(g, rows[:4], want_mcn=True)
    assert not F.any() and not Fo.any() and M[:4].tolist() == Mo.tolist() == [1, 1, 1, 0]
    assert np.array_equal(M, np.tile(M[:4], 513))
