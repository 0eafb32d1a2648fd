"""GPU parity of the 16-bit filters' workgroup units above 64 dimensions (K padded
to 80 and 96, and 112 beside them): units with every remainder of a wave's 64
queries, chunks of 64 candidates cut in either half, the minimum of a tile first
and the direct scan.  Pair lists must equal the oracle's."""
import numpy as np
import pytest

import datagen
import oracle
from test_gpu_parity import assert_same_as_oracle, calibrated
from test_gpu_query import gpu_query_join

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def one_cell(n, d, seed):
    P = datagen.offgrid("uniform64", n, d, seed=seed)
    P[:, 0] *= np.float32(2.0 ** -12)  # the indexed dimension
    return P


@pytest.mark.parametrize("hits", ["0", "1"])
@pytest.mark.parametrize("n", [193, 225, 256, 449, 1025, 1249])
@pytest.mark.parametrize("d,prec", [(65, "fp16"), (80, "bf16"), (81, "bf16"), (90, "fp16"),
                                    (96, "fp16"), (97, "fp16")])
def test_edges(n, d, prec, hits, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_HITS", hits)
    P = one_cell(n, d, 980 + n + d)
    eps = calibrated(P, 20, stride=3)
    print("case wide16", n, d, prec, hits, flush=True)
    info = assert_same_as_oracle(P, eps, precision=prec, k=1, reorder=0)
    assert info["units"] == 1 and info["n_cells"] == 1


@pytest.mark.parametrize("m,d", [(225, 70), (449, 90)])
def test_query_join(m, d):
    E, Q = one_cell(1249, d, 990), one_cell(m, d, 991)
    eps = calibrated(E, 20, stride=3)
    print("case wide16 query", m, d, flush=True)
    gi, gj, _, info, _ = gpu_query_join(Q, E, eps, precision="bf16", k=1, reorder=0)
    assert info["units"] == 1
    oi, oj = oracle.join(Q, E, eps)
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)
