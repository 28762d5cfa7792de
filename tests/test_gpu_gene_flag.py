"""The gene check of checked calls sees their own rows alone: trusted rows with a
gene that is no node, still running on another stream while a checked call is
answered, leave the next checked call as it is."""
import numpy as np
import pytest

from oracle import cnd_oracle as O
from paper_2412_20980_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["eval", "sixdst"])
def test_trusted_rows_on_another_stream(which):
    import torch
    from paper_2412_20980_amd import gapa
    g = inputs.barabasi_albert(300, 2, seed=4)
    rows = inputs.random_population(g.n, 9, 6, seed=2)
    good = torch.from_numpy(rows).cuda()
    bad = good.clone()
    bad[2, 1] = g.n
    graph = gapa.Graph.from_csr(g)

    def call(genes, trust, stream=None):
        if which == "eval":
            return graph.eval(genes, trust=trust, stream=stream)
        return graph.sixdst(genes, g.n, trust=trust, stream=stream)[0]

    call(good, False)
    other = torch.cuda.Stream()
    with torch.cuda.stream(other):
        torch.cuda._sleep(200_000_000)  # the trusted rows start after the next checked call
        call(bad, True, other)
    F = call(good, False)
    assert not other.query()
    torch.cuda.synchronize()
    again = call(good, False)
    with pytest.raises(gapa.GapaError) as e:
        call(bad, False)
    assert e.value.code == gapa.GAPA_E_BAD_GENE
    want = O.eval_population(g, rows)
    for f in (F, again, call(good, False)):
        assert np.array_equal(f.cpu().numpy(), want)
