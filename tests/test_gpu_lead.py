"""GPU parity of the FP32 matrix-core joins with their tiles' leading products first
and with all products at once: every K padding behind the query box and some above,
units and parts cut at every remainder, norms far above eps (most tiles pass the
leading product) and partners within rounding of eps.  Pair lists must equal the
oracle's."""
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


@pytest.fixture(params=["0", "1"], autouse=True)
def lead(request, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_LEAD", request.param)
    return request.param


@pytest.mark.parametrize("n", [4353, 4415])
@pytest.mark.parametrize("d", [9, 16, 17, 24, 31, 40, 90])
def test_dimensions(n, d, lead):
    P = datagen.offgrid("uniform64", n, d, seed=1000 + n + d)
    print("case lead", n, d, lead, flush=True)
    info = assert_same_as_oracle(P, calibrated(P, 20, stride=9), k=1)
    assert info["candidates"] >= 2 ** 24 and info["fp32_form"] == 2


@pytest.mark.parametrize("d", [12, 20, 40])
def test_norms_far_above_the_radius(d, lead):
    """eps^2 below 2^-10 of the squared norms: the leading product rejects little."""
    base = datagen.offgrid("uniform64", 3000, d, seed=1040 + d)
    rng = np.random.default_rng(1041 + d)
    near = base[rng.integers(0, len(base), 1600)]
    near = (near + 1e-3 * rng.standard_normal(near.shape)).astype(np.float32)
    P = np.concatenate([base, near])
    P[:, 0] *= np.float32(1e-3)  # the indexed dimension: two cells
    print("case lead norms", d, lead, flush=True)
    info = assert_same_as_oracle(P, 5e-3, k=1, reorder=0)
    assert info["fp32_form"] == 2


@pytest.mark.parametrize("d,opts", [(16, dict(min_batches=3)), (24, dict(batch_pairs=20000)),
                                    (16, dict(sortidu=True)), (40, dict(min_batches=3))])
def test_partners_and_options(d, opts, lead):
    base = datagen.offgrid("normal_binades", 3700, d, seed=1060 + d)
    eps = calibrated(base, 8, stride=9)
    P = np.concatenate([base, datagen.partners_near_radius(base, eps, 900, seed=1070 + d)])
    print("case lead options", d, opts, lead, flush=True)
    assert_same_as_oracle(P, eps, k=1, **opts)
