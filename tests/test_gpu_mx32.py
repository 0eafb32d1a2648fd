"""GPU parity of the FP32 filter on the matrix cores: joins of at least 2^24
candidate pairs whose 256-query units are mostly full take it.  Pair lists
must equal the oracle's exactly; distances are checked at 1e-5 relative.

Sizes: every padded dimension the kernel is instantiated for and its edges
(8, 16 / 17 .. 24 / 25 .. 32 / 33 .. 48 / .. / 128), candidate counts that
are no multiple of the 32-column tile, units with one query past a block."""
import numpy as np
import pytest

import datagen
import oracle
from test_gpu_parity import assert_same_as_oracle, calibrated, gpu_join
from test_gpu_query import gpu_query_join

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("d", [1, 3, 8, 16, 17, 24, 25, 32, 33, 48, 49, 64, 65, 90, 97, 112, 113,
                               128])
def test_every_padded_dimension(d):
    # few dimensions: a radius and k that leave at least 2^24 candidates
    n = 4353 if d > 8 else 9001  # 17 x 256 + 1
    P = datagen.uniform_grid(n, d, 200 + d)
    eps = {1: 0.125, 3: 0.2}.get(d) or calibrated(P, 20, stride=9)
    print("case mx32 uniform", d, flush=True)
    info = assert_same_as_oracle(P, eps, k=1 if d <= 8 else 0)
    assert info["candidates"] >= 2 ** 24 and info["fp32_form"] == 2 and info["units"] == 1


@pytest.mark.parametrize("n,d,centres", [(12000, 18, 3), (9000, 40, 4), (10000, 90, 5)])
def test_clusters(n, d, centres):
    """Clusters far apart (the ball and box tests reject whole clusters), off
    the coarse grid."""
    std = datagen.uniform_std(d, 0.01, 0.05, 300 + d)
    rng = np.random.default_rng(301 + d)
    c = rng.random((centres, d)) * 3.0 + 100.0
    P = (c[rng.integers(0, centres, n)] + rng.standard_normal((n, d)) * std).astype(np.float32)
    print("case mx32 clusters", d, flush=True)
    info = assert_same_as_oracle(P, calibrated(P, 30, stride=17))
    assert info["fp32_form"] == 2


@pytest.mark.parametrize("d", [6, 24, 30, 70])
def test_partners_at_radius(d):
    """Partners within a few float32 roundings of eps reach the FP64 recheck."""
    base = datagen.offgrid("normal_binades", 3600, d, seed=400 + d)
    eps = calibrated(base, 8, stride=9)
    P = np.concatenate([base, datagen.partners_near_radius(base, eps, 900, seed=410 + d),
                        datagen.partners_near_radius(base, eps, 500, seed=420 + d,
                                                     unit=2.0 ** -23)])
    print("case mx32 partners", d, flush=True)
    assert assert_same_as_oracle(P, eps, k=1)["rechecks"] > 0


def test_duplicates_and_exact_ties():
    u = 2.0 ** -24
    ties = np.array([[0, 0, 0, 0], [3000 * u, 4000 * u, 0, 0], [3000 * u, 3999 * u, 89 * u, 0],
                     [3000 * u, 4000 * u, u, 0]], dtype=np.float32)
    spread = (datagen.uniform_grid(4500, 4, 31) * np.float32(0.0005)).astype(np.float32)
    P = np.concatenate([ties, np.repeat(spread[:100], 3, axis=0), spread])
    info = assert_same_as_oracle(P, 5000 * u, k=2)
    assert info["candidates"] >= 2 ** 24


@pytest.mark.parametrize("d", [10, 40])
@pytest.mark.parametrize("opts", [dict(min_batches=3), dict(sortidu=True), dict(batch_pairs=40000)])
def test_options(d, opts):
    P = datagen.offgrid("uniform64", 4700, d, seed=500 + d)
    print("case mx32 options", d, opts, flush=True)
    assert_same_as_oracle(P, calibrated(P, 15, stride=9), **opts)


@pytest.mark.parametrize("opts", [dict(), dict(min_batches=3)])
def test_undersized_buffers(opts, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_UNDERSIZE", "1")
    P = datagen.uniform_grid(4500, 12, 61)
    assert_same_as_oracle(P, calibrated(P, 25, stride=9), **opts)


@pytest.mark.parametrize("m,d", [(4300, 12), (4100, 50), (7, 12)])
def test_query_join(m, d):
    """Queries partly outside E's range; seven queries stay on the vector
    path of an index built for the matrix cores."""
    E = datagen.offgrid("uniform64", 4600, d, seed=600 + d)
    Q = datagen.offgrid("uniform64", m, d, seed=601 + d)
    Q[: m // 5] += np.float32(0.4)
    eps = calibrated(E, 15, stride=9)
    print("case mx32 query", m, d, flush=True)
    gi, gj, gd, info, _ = gpu_query_join(Q, E, eps)
    oi, oj, os_ = oracle.join(Q, E, eps, with_dist=True)
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)
    np.testing.assert_allclose(gd, np.sqrt(os_), rtol=1e-5, atol=1e-30)


@pytest.mark.parametrize("log2_scale", [-32, 41])
def test_scaled_data(log2_scale):
    """Powers of two scale coordinates and radius: the pairs stay the same."""
    P = datagen.uniform_grid(4400, 12, 71)
    eps = calibrated(P, 20, stride=9)
    s = 2.0 ** log2_scale
    a = gpu_join(P, eps)
    b = gpu_join((P * np.float32(s)).astype(np.float32), eps * s)
    assert a[3]["candidates"] >= 2 ** 24
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("d,far,form", [(40, 2.0 ** 9, 2), (40, 2.0 ** 17, 1)])
def test_outliers(d, far, form):
    """A few points far from the rest set the scale of the split rows; past
    2^15 radii the join keeps the vector form (difference above 16 dimensions)."""
    P = datagen.offgrid("uniform64", 4500, d, seed=700 + d)
    P[:3] *= np.float32(far)
    eps = calibrated(P, 20, stride=9)
    print("case mx32 outliers", d, far, flush=True)
    assert assert_same_as_oracle(P, eps)["fp32_form"] == form
