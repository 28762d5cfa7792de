"""Fitness of graphs too large for one workgroup and without hubs, where further
rounds follow the sweeps, through the C ABI against the oracle: random graphs
around their critical degree, a tree, a path and a lattice (which stop early), a
power law (no rounds), for one individual, one word and several words a node;
the allocation-free entry point, a GA and a batch with such a graph."""
import numpy as np
import pytest

from oracle import cnd_oracle as O
from paper_2412_20980_amd import inputs

pytestmark = pytest.mark.gpu
N = 66_000


@pytest.fixture(scope="module")
def gp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2412_20980_amd import gapa
    return gapa


def graph_of(kind):
    p = np.random.default_rng(1).permutation(N)
    if kind == "path":
        return inputs.csr_from_edges(N, p[:-1], p[1:])
    if kind == "lattice":
        i = p.reshape(264, 250)
        return inputs.csr_from_edges(N, np.concatenate([i[:, :-1].ravel(), i[:-1].ravel()]),
                                     np.concatenate([i[:, 1:].ravel(), i[1:].ravel()]))
    if kind == "tree":
        return inputs.barabasi_albert(N, 1, seed=3)
    if kind == "power":
        return inputs.chung_lu(N, 2.5, 8.0, 260_000, seed=7)
    return inputs.erdos_renyi(N, float(kind), seed=4)


@pytest.mark.parametrize("kind", ["1.2", "2.0", "4.0", "8.0", "tree", "path", "lattice", "power"])
@pytest.mark.parametrize("P", [1, 40, 300])
def test_fitness_matches_oracle(gp, kind, P):
    import torch
    g = graph_of(kind)
    rows = inputs.random_population(N, 600, P, seed=P)
    print(f"{kind} P={P}", flush=True)
    graph = gp.Graph.from_csr(g)
    fit, mcn = graph.eval(rows, want_mcn=True)
    ref, ref_mcn = O.eval_population(g, rows, want_mcn=True)
    assert np.array_equal(fit, ref) and np.array_equal(mcn, ref_mcn)
    d = torch.from_numpy(rows).cuda()
    for _ in range(2):
        f = gp.gapa_eval_population_noalloc(graph.handle, d)
        assert np.array_equal(f.cpu().numpy(), ref)


def test_ga_and_batch_match_oracle(gp):
    g, small = graph_of("3.0"), inputs.erdos_renyi(900, 2.0, seed=5)
    graphs = [gp.Graph.from_csr(x) for x in (g, small)]
    params = [dict(k=500, pop=20, seed=3), dict(k=9, pop=33, seed=4)]
    single = gp.GA(graphs[0], replay=True, **params[0])
    batch = gp.Batch(graphs, params)
    refs = [O.OracleGA(x, **p) for x, p in zip((g, small), params)]
    for gen in range(4):
        pop, F = single.population()
        assert np.array_equal(F, refs[0].F) and np.array_equal(pop, refs[0].pop), gen
        for b, r in enumerate(refs):
            pop, F = batch.population(b)
            assert np.array_equal(F, r.F) and np.array_equal(pop, r.pop), (gen, b)
        single.step(1)
        batch.step(1)
        for r in refs:
            r.step()


@pytest.mark.parametrize("P", [1, 33, 128, 129, 256, 257])
@pytest.mark.parametrize("hubs", [0.0, 0.9])
def test_sparse_graph_with_hubs_matches_oracle(gp, hubs, P):
    # rounds where the sweeps still gain (hubs removed), none where they do not;
    # one to eight words a node, and sixteen (no such launch)
    import torch
    g = inputs.barabasi_albert(70_000, 2, seed=6)
    rows = inputs.hub_biased_population(g, 900, P, seed=P, hub_frac=hubs) if hubs else \
        inputs.random_population(g.n, 900, P, seed=P)
    print(f"hubs={hubs} P={P}", flush=True)
    graph = gp.Graph.from_csr(g)
    fit, mcn = graph.eval(rows, want_mcn=True)
    ref, ref_mcn = O.eval_population(g, rows, want_mcn=True)
    assert np.array_equal(fit, ref) and np.array_equal(mcn, ref_mcn)
    d = torch.from_numpy(rows).cuda()
    f = gp.gapa_eval_population_noalloc(graph.handle, d)
    assert np.array_equal(f.cpu().numpy(), ref)
