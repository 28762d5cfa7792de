"""gapa_eval_population_noalloc maps no memory, on a handle's first checked call
either: the process's mappings of the GPU driver (device memory and page-locked
host memory alike) are the same before and after.  Handles that hold the
page-locked memory of host-array calls, more of them than the library keeps
spare, see to it that none is lying ready."""
import numpy as np
import pytest

from oracle import cnd_oracle as O
from paper_2412_20980_amd import inputs

pytestmark = pytest.mark.gpu


def driver_mappings():
    with open("/proc/self/maps") as f:
        return sorted(line.split()[0] for line in f if "/dev/dri/" in line or "/dev/kfd" in line)


def test_first_checked_call_of_a_handle_maps_nothing():
    import torch
    from paper_2412_20980_amd import gapa
    g = inputs.barabasi_albert(500, 2, seed=8)
    genes = inputs.random_population(g.n, 10, 4, seed=9)
    d = torch.from_numpy(genes).cuda()
    bad = d.clone()
    bad[1, 2] = g.n
    fit = torch.empty(4, dtype=torch.int64, device="cuda")
    holders = [gapa.Graph.from_csr(g) for _ in range(12)]
    for h in holders:
        h.eval(genes)
    gapa.gapa_eval_population_noalloc(holders[0].handle, d, fitness=fit)  # kernels loaded
    fresh = gapa.Graph.from_csr(g)
    before = driver_mappings()
    assert before
    gapa.gapa_eval_population_noalloc(fresh.handle, d, fitness=fit)
    with pytest.raises(gapa.GapaError) as e:
        gapa.gapa_eval_population_noalloc(fresh.handle, bad, fitness=fit)
    after = driver_mappings()
    assert e.value.code == gapa.GAPA_E_BAD_GENE
    gapa.gapa_eval_population_noalloc(fresh.handle, d, fitness=fit)
    assert np.array_equal(fit.cpu().numpy(), O.eval_population(g, genes))
    assert after == before
