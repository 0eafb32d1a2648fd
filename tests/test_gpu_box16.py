"""GPU parity of the 16-bit filters' query-box kernel at the edges of its tiles:
parts of a unit with one query, the last block of candidates cut at every
remainder, K padded to 16 and 32, few and many hits per tile, and result
batches that skip earlier candidates.  Pair lists must equal the oracle's."""
import numpy as np
import pytest

import datagen
from test_gpu_parity import assert_same_as_oracle, calibrated

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.fixture(autouse=True)
def box_form(monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_BOX", "1")


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("d", [1, 7, 8, 9, 16, 17, 24, 32])
@pytest.mark.parametrize("n", [1, 31, 257, 1025])
def test_edges(n, d, prec):
    P = datagen.offgrid("uniform64", n, d, seed=600 + n + d)
    eps = calibrated(P, min(12, n / 4), stride=1) if n > 31 else 0.3
    print("case box16", n, d, prec, flush=True)
    assert_same_as_oracle(P, eps, k=1, precision=prec)


@pytest.mark.parametrize("target", [2, 700])
@pytest.mark.parametrize("opts", [dict(), dict(min_batches=3), dict(sortidu=True)])
def test_selectivities_and_options(target, opts):
    P = datagen.offgrid("mixture_f32", 4133, 16, seed=640)
    print("case box16 options", target, opts, flush=True)
    assert_same_as_oracle(P, calibrated(P, target, stride=5), precision="fp16", k=2, **opts)
