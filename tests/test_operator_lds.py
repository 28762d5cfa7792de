"""LDS of the operator kernels at the limit of a compute unit (CPU only): sizes
that are let through fit with what the kernels declare besides, and every size
whose sets alone (unpadded) leave 72 bytes is let through."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIMIT, STATIC = 160 * 1024, 48


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    exe = tmp_path_factory.mktemp("lds") / "operator_lds"
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", f"-I{ROOT}/include",
                    f"-I{ROOT}/paper_2412_20980_amd/csrc", os.path.join(HERE, "operator_lds.cpp"), "-o", str(exe)],
                   check=True, cwd="/tmp")

    def run(sizes):
        text = "\n".join(f"{n} {k}" for n, k in sizes)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return np.array([line.split() for line in out.splitlines()], dtype=np.int64)
    return run


def sets_bytes(n, k):
    """Membership bits, the row, its slot list and three bit sets over the slots."""
    return 4 * ((n + 31) // 32 + k + 3 * ((k + 31) // 32)) + 2 * ((k + 1) // 2 * 2)


def test_sizes_at_the_limit(layout):
    sizes = [(290720, 20000), (290336, 20000), (1_305_000, 3), (1_310_720, 1), (60000, 30000)]
    rng = np.random.default_rng(3)
    for k in [1, 2, 3, 30, 31, 32, 33, 1000] + rng.integers(2, 26000, 200).tolist():
        # the graphs whose sets come to the limit, a few words less or more
        n = 32 * ((LIMIT - sets_bytes(0, k)) // 4)
        sizes += [(n - d, k) for d in [0, 1, 31, 32, 33, 64, 96, 100, 128, 256, 384, 512, 576, 608, 640, 1000, 4096]
                  if 2 * k <= n - d]
    got = layout(sizes)
    assert got.shape == (len(sizes), 3) and len(sizes) > 1000
    for (n, k), (lds, log_q, ok) in zip(sizes, got.tolist()):
        words = -(-n // 128) * 4
        quads = -(-words // (1 << log_q))
        # the layout as the kernels carve it
        need = 4 * (words + k + 3 * ((k + 31) // 32)) + 2 * max(k, quads)
        assert need <= lds and ok == (lds + STATIC <= LIMIT), (n, k)
        if sets_bytes(n, k) + 72 <= LIMIT:
            assert ok, (n, k)
    assert got[0, 2] == 0 and got[1, 2] == 0 and got[:, 2].sum() > 100


@pytest.mark.gpu
def test_gas_at_the_limit():
    from oracle import cnd_oracle as O
    from paper_2412_20980_amd import gapa, inputs
    k = 20000
    for n, fits in ((290_304, True), (290_336, False), (290_720, False)):
        u = np.arange(n - 1)
        g = inputs.csr_from_edges(n, u, u + 1)
        print(f"path n={n} k={k}", flush=True)
        graph = gapa.Graph.from_csr(g, trust=True)
        if not fits:
            with pytest.raises(gapa.GapaError) as e:
                gapa.GA(graph, k, 3, 5)
            assert e.value.code == gapa.GAPA_E_INVALID_ARG
            continue
        ga, ref = gapa.GA(graph, k, 3, 5), O.OracleGA(g, k, 3, 5)
        ga.step(1)
        ref.step()
        rows, F = ga.population()
        assert np.array_equal(rows, ref.pop) and np.array_equal(F, ref.F)
