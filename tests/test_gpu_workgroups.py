"""Fitness by one workgroup for every few individuals (graphs of at most 65,535
nodes), through the C ABI, at the sizes where its shape changes: threads of a
block, individuals to a block (one to eight, with four to a state byte or
eight), the node counts at which the states leave less LDS for leftover
nodes or none, populations that do not fill the last block; graphs without
edges, with isolated nodes, with hubs and without, trees and paths whose
leftover nodes outgrow LDS; rows that remove everything, nothing, or repeat a
gene.  Every row against the library's edge-parallel union-find, a sample
against the oracle; exact integers."""
import numpy as np
import pytest

from oracle import cnd_oracle as O
from paper_2412_20980_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2412_20980_amd import gapa
    return gapa


def graph_of(kind, n):
    if kind == "path":
        v = np.random.default_rng(n).permutation(n)
        return inputs.csr_from_edges(n, v[:-1], v[1:])
    if kind == "tree":
        return inputs.barabasi_albert(n, 1, seed=n)
    if kind == "ba":
        return inputs.barabasi_albert(n, 2, seed=n)
    if kind == "star":
        return inputs.csr_from_edges(n, np.zeros(n - 1, dtype=np.int64), np.arange(1, n))
    if kind == "empty":
        return inputs.csr_from_edges(n, np.zeros(0, dtype=np.int64), np.zeros(0, dtype=np.int64))
    return inputs.erdos_renyi(n, float(kind), seed=n)  # mean degree


def rows_of(g, P, seed):
    """P rows of n / 50 genes: hubs and others, one in ten with a repeated gene."""
    rng = np.random.default_rng(seed)
    k = min(g.n, max(2, g.n // 50))  # (a row has at most n genes)
    top = np.argsort(-g.degrees(), kind="stable")[:3 * k]
    rows = np.concatenate([rng.choice(top, size=(P, k // 2)), rng.integers(0, g.n, size=(P, k - k // 2))], axis=1)
    rows[::10, -1] = rows[::10, 0]
    return rows.astype(np.int32)


@pytest.mark.parametrize("kind,n,P", [
    ("empty", 1, 3), ("empty", 40, 9), ("1.0", 33, 100), ("ba", 512, 1025), ("2.0", 513, 512), ("ba", 4096, 513),
    ("3.0", 4097, 257), ("ba", 4097, 1025), ("8.0", 5000, 1), ("star", 9000, 300), ("tree", 9000, 520),
    ("path", 3000, 600), ("path", 18000, 40), ("path", 18001, 40), ("1.5", 20000, 2050), ("tree", 40000, 1030),
    ("6.0", 40001, 1030), ("tree", 60000, 70), ("4.0", 65535, 300), ("4.0", 65536, 40)])
def test_shapes_match_union_find_and_oracle(gp, kind, n, P):
    g = graph_of(kind, n)
    rows = rows_of(g, P, seed=n + P)
    print(f"{kind} n={n} P={P}", flush=True)
    a, b = gp.Graph.from_csr(g), gp.Graph.from_csr(g, unionfind=True)
    F, M = a.eval(rows, want_mcn=True)
    Fu, Mu = b.eval(rows, want_mcn=True)
    assert np.array_equal(F, Fu) and np.array_equal(M, Mu)
    assert np.array_equal(a.eval(rows, objective="components"), b.eval(rows, objective="components"))
    idx = np.unique(np.linspace(0, P - 1, 6).astype(int))
    Fo, Mo = O.eval_population(g, rows[idx], want_mcn=True)
    assert np.array_equal(F[idx], Fo) and np.array_equal(M[idx], Mo)


def test_everything_and_nothing_removed(gp):
    g = inputs.erdos_renyi(300, 1.5, seed=5)  # a fifth of the nodes are isolated
    iso = np.flatnonzero(g.degrees() == 0)
    assert iso.size > 10
    graph = gp.Graph.from_csr(g)
    every = np.arange(g.n, dtype=np.int32)
    but_one = np.where(every == iso[0], every[every != iso[0]][0], every).astype(np.int32)
    F, M = graph.eval(np.stack([every, but_one]), want_mcn=True)
    assert F.tolist() == [0, 0] and M.tolist() == [0, 1]  # nothing survives; one isolated node does
    F, M = graph.eval(np.zeros((9, 0), dtype=np.int32), want_mcn=True)
    Fo, Mo = O.pc(g, [])
    assert (F == Fo).all() and (M == Mo).all()


def test_noalloc_and_ga_take_the_same_way(gp):
    """The allocation-free entry point and a GA's generations (MCN objective,
    and a population that changes the individuals of a block) on graphs whose
    leftover nodes outgrow LDS."""
    import torch
    g = graph_of("tree", 30000)
    graph = gp.Graph.from_csr(g)
    rows = rows_of(g, 300, seed=3)
    d = torch.from_numpy(rows).cuda()
    f, m = gp.gapa_eval_population_noalloc(graph.handle, d, flags=gp.GAPA_WANT_MCN)
    F, M = gp.Graph.from_csr(g, unionfind=True).eval(rows, want_mcn=True)
    assert np.array_equal(f.cpu().numpy(), F) and np.array_equal(m.cpu().numpy(), M)
    small = inputs.barabasi_albert(1500, 2, seed=9)
    ga = gp.GA(gp.Graph.from_csr(small), 20, 70, seed=4, offspring=600, objective="mcn", replay=True)
    ref = O.OracleGA(small, 20, 70, 4, offspring=600, objective="mcn")
    for _ in range(4):
        ga.step(1)
        ref.step()
    pop, F = ga.population()
    assert np.array_equal(pop, ref.pop) and np.array_equal(F, ref.F)


@pytest.mark.parametrize("kind,n,k,P,lam,objective", [
    ("ba", 1000, 60, 20, 256, "mcn"),          # as many children as workgroups
    ("ba", 5000, 60, 20, 257, "components"),   # one more: workgroups of several, bred apart
    ("path", 45000, 700, 6, 0, "components"),  # a graph the bit-parallel pass keeps
    ("tree", 30000, 900, 9, 12, "pc"),
    ("3.0", 48500, 24000, 3, 0, "pc"),         # the operators need more LDS than the evaluation
])
def test_children_bred_in_place_follow_the_oracle(gp, kind, n, k, P, lam, objective):
    g = graph_of(kind, n)
    print(f"{kind} n={n} k={k} P={P} lambda={lam} {objective}", flush=True)
    graph = gp.Graph.from_csr(g)
    ga = gp.GA(graph, k, P, 21, 0.6, 0.1, 3, lam, objective=objective)
    timed = gp.GA(graph, k, P, 21, 0.6, 0.1, 3, lam, objective=objective)
    timed.set_timing(True)
    oga = O.OracleGA(g, k, P, 21, 0.6, 0.1, 3, lam, objective=objective)
    for gen in range(4):
        for x in (ga, timed):
            pop, F = x.population()
            assert np.array_equal(F, oga.F) and np.array_equal(pop, oga.pop), gen
            x.step(1)
        oga.step()


@pytest.mark.parametrize("kind,n,k,P,lam,objective", [
    ("ba", 200, 10, 32, 0, "pc"),
    ("2.0", 60, 1, 1, 255, "pc"),            # one parent; as many keys as threads
    ("2.0", 60, 2, 200, 56, "components"),   # more rows to copy than blocks; many equal keys
    ("empty", 40, 3, 9, 12, "components"),   # all keys equal
    ("3.0", 900, 30, 128, 128, "pc"),
    ("3.0", 900, 30, 128, 129, "pc"),        # one key too many: elitism launched by itself
    ("tree", 30000, 900, 9, 12, "pc"),
    ("1.5", 2500, 700, 40, 20, "mcn"),       # an objective of its own launch
])
def test_generations_of_one_call_follow_the_oracle(gp, kind, n, k, P, lam, objective):
    """Calls of one, two and more generations, in every parity, the children's
    buffers swapped in between; timing on for one call, some recorded."""
    g = graph_of(kind, n)
    print(f"{kind} n={n} k={k} P={P} lambda={lam} {objective}", flush=True)
    graph = gp.Graph.from_csr(g)
    ga, replayed = (gp.GA(graph, k, P, 22, 0.6, 0.1, 2, lam, replay=r, objective=objective) for r in (False, True))
    oga = O.OracleGA(g, k, P, 22, 0.6, 0.1, 2, lam, objective=objective)
    for steps, timing in ((2, 0), (1, 0), (3, 0), (5, 0), (2, 1), (4, 0), (5, 0), (5, 0)):
        if steps == 5:
            replayed.record(5)
        for _ in range(steps):
            oga.step()
        for x in (ga, replayed):
            x.set_timing(timing)
            x.step(steps)
            pop, F = x.population()
            assert np.array_equal(F, oga.F) and np.array_equal(pop, oga.pop), steps
            genes, f, gens = x.best()
            assert gens == oga.generation and f == oga.F[0] and np.array_equal(genes, oga.pop[0])


@pytest.mark.parametrize("kinds", [
    [("tree", 30000, 40), ("ba", 400, 100), ("2.0", 41000, 33), ("empty", 5, 7), ("3.0", 3000, 128)],
    [("ba", 300, 9), ("star", 500, 70)],
    [("4.0", 65536, 20), ("ba", 900, 50)]])  # one graph too large: the bit-parallel pass takes the batch
def test_batches_follow_single_gas(gp, kinds):
    graphs = [graph_of(kind, n) for kind, n, _ in kinds]
    params = [dict(k=max(1, g.n // 60), pop=P, seed=5 + b, offspring=P + 10 * b)
              for b, (g, (_, _, P)) in enumerate(zip(graphs, kinds))]
    handles = [gp.Graph.from_csr(g) for g in graphs]
    print(kinds, flush=True)
    bt = gp.Batch(handles, params)
    gas = [gp.GA(h, **p) for h, p in zip(handles, params)]
    for h in handles:
        h.close()  # the batch and the GAs keep what they need
    bt.step(5)
    for b, ga in enumerate(gas):
        ga.step(5)
        (rows, F), (rows1, F1) = bt.population(b), ga.population()
        assert np.array_equal(F, F1) and np.array_equal(rows, rows1), b
        Fo = O.eval_population(graphs[b], rows[:4])
        assert np.array_equal(F[:4], Fo), b


@pytest.mark.parametrize("arcs", [[], [(0, 1)], [(0, 1), (1, 2), (2, 0)]])
def test_repeated_arcs_of_a_trusted_graph(gp, arcs):
    """Arcs that a trusted CSR holds twice one way only (one list has no room
    for it; every list has, but with other ids) change no component."""
    g = inputs.barabasi_albert(2500, 3, seed=2)
    g = inputs.csr_from_edges(g.n, np.concatenate([np.repeat(np.arange(g.n), g.degrees()), [0, 1, 2]]),
                              np.concatenate([g.col_idx, [1, 2, 0]]))
    lists = [list(g.col_idx[g.row_ptr[v]:g.row_ptr[v + 1]]) for v in range(g.n)]
    for u, v in arcs:
        lists[u] = sorted(lists[u] + [v])
    rp = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)
    graph = gp.Graph(g.n, rp, np.concatenate(lists).astype(np.int32), trust=True)
    rows = inputs.random_population(g.n, 200, 40, seed=9)
    assert np.array_equal(graph.eval(rows), O.eval_population(g, rows))
