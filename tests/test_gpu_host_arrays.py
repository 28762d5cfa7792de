"""Calls with host arrays, through the C ABI: results equal those of the same
call on device arrays (and the device's own population), on both sides of the
sizes at which the arrays stop passing through page-locked memory (512 KiB of
genes, 1 MiB of results), with more handles than spare page-locked buffers, and
from several threads; a bad gene is still refused after good calls."""
import threading

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


@pytest.mark.parametrize("P,k", [(1, 0), (1, 1), (1024, 128), (1024, 129), (90_000, 1)])
def test_eval_equals_device_arrays(gp, P, k):
    import torch
    g = inputs.erdos_renyi(500, 2.0, seed=3)
    graph = gp.Graph.from_csr(g)
    genes = inputs.random_population(g.n, k, P, seed=P + k) if k else np.zeros((P, 0), dtype=np.int32)
    print(f"P={P} k={k}", flush=True)
    f, m = graph.eval(genes, want_mcn=True)
    fd, md = graph.eval(torch.from_numpy(genes).cuda(), want_mcn=True)
    assert np.array_equal(f, fd.cpu().numpy()) and np.array_equal(m, md.cpu().numpy())
    for i in (0, P - 1):
        assert (int(f[i]), int(m[i])) == O.pc(g, genes[i])
    if k:
        bad = torch.from_numpy(genes).cuda()
        bad[P - 1, k - 1] = g.n
        with pytest.raises(gp.GapaError):
            graph.eval(bad)
        assert np.array_equal(graph.eval(genes), f)


@pytest.mark.parametrize("P,k", [(4, 3), (1000, 259), (1000, 260), (2000, 300)])
def test_population_follows_the_oracle(gp, P, k):
    g = inputs.erdos_renyi(700, 3.0, seed=4)
    graph = gp.Graph.from_csr(g)
    gas = [gp.GA(graph, k, P, seed) for seed in range(12 if P == 4 else 1)]
    for seed, ga in enumerate(gas):
        ga.step(1)
        oga = O.OracleGA(g, k, P, seed)
        oga.step()
        pop, F = ga.population()
        assert np.array_equal(pop, oga.pop) and np.array_equal(F, oga.F)
        genes, f, gens = ga.best()
        assert gens == 1 and f == oga.F[0] and np.array_equal(genes, oga.pop[0])


def test_threads(gp):
    wrong = []

    def work(seed):
        g = inputs.barabasi_albert(300 + seed, 2, seed=seed)
        for rep in range(4):
            graph = gp.Graph.from_csr(g)
            genes = inputs.random_population(g.n, 9, 40, seed=seed + rep)
            if not np.array_equal(graph.eval(genes), O.eval_population(g, genes, nthreads=1)):
                wrong.append((seed, rep))
            graph.close()

    threads = [threading.Thread(target=work, args=(s,)) for s in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
