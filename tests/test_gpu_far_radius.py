"""GPU parity of the 16-bit filters at radii whose squares pass the FP32 range:
every pair is a result, thresholds saturate, and blocks of 32 candidates and
queries with fewer rows must add nothing.  Pair lists must equal the oracle's."""
import numpy as np
import pytest

import datagen
import oracle
from test_gpu_parity import assert_same_as_oracle
from test_gpu_query import gpu_query_join

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("box,hits", [("0", "0"), ("0", "1"), ("1", "0")])
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("n,d", [(1, 8), (33, 16), (225, 24), (289, 70)])
def test_every_pair(n, d, prec, box, hits, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_BOX", box)
    monkeypatch.setenv("SJ_DEBUG_HITS", hits)
    P = datagen.offgrid("uniform64", n, d, seed=800 + n)
    print("case far radius", n, d, prec, box, hits, flush=True)
    info = assert_same_as_oracle(P, 1e20, precision=prec)
    assert info["pairs"] == n * n


@pytest.mark.parametrize("m", [1, 40, 225])
def test_every_query_pair(m):
    E = datagen.offgrid("uniform64", 289, 16, seed=810)
    Q = datagen.offgrid("uniform64", m, 16, seed=811)
    print("case far radius query", m, flush=True)
    gi, gj = gpu_query_join(Q, E, 1e20, precision="bf16")[:2]
    oi, oj = oracle.join(Q, E, 1e20)
    assert len(oi) == m * len(E)
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)
