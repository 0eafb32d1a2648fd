"""GPU parity of the group test of the FP32 joins above 24 dimensions: pivots at
equal distances and picked ones (from 16384 points on), clusters with and without a
pivot of their own, more clusters than directions, points in a subspace of few
dimensions, units with few queries.  Pair lists must equal the oracle's."""
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


def clusters(n, d, centres, seed, rare=False):
    rng = np.random.default_rng(seed)
    c = rng.random((centres, d)) * 2.0 - 7.0
    label = rng.integers(0, centres, n)
    if rare:  # one cluster of nine points
        label = np.where(label == 0, 1, label)
        label[rng.permutation(n)[:9]] = 0
    std = datagen.uniform_std(d, 0.01, 0.2, seed + 1)
    return (c[label] + rng.standard_normal((n, d)) * std).astype(np.float32)


@pytest.mark.parametrize("n", [16383, 16384, 16385])
@pytest.mark.parametrize("d,centres,rare", [(26, 20, False), (90, 20, True), (128, 70, False)])
def test_clusters(n, d, centres, rare):
    P = clusters(n, d, centres, 900 + d, rare)
    print("case groups", n, d, centres, flush=True)
    info = assert_same_as_oracle(P, calibrated(P, 20, stride=97), k=2)
    assert info["fp32_form"] == 2


@pytest.mark.parametrize("rank", [0, 3, 33])
def test_flat_sets(rank):
    """Points of a plane of few dimensions (rank 0: copies of few points)."""
    rng = np.random.default_rng(930 + rank)
    P = rng.random((17000, rank)) @ rng.random((rank, 40)) if rank else \
        rng.random((60, 40))[rng.integers(0, 60, 17000)]
    P = np.ascontiguousarray(P.astype(np.float32))
    # (some pivots equal, some directions from the axes)
    print("case groups flat", rank, flush=True)
    assert_same_as_oracle(P, calibrated(P, 20, stride=97) if rank else 0.01, k=2)


@pytest.mark.parametrize("opts", [dict(min_batches=5), dict(batch_pairs=60000)])
def test_batches(opts):
    P = clusters(16500, 37, 12, 950)
    print("case groups batches", opts, flush=True)
    assert_same_as_oracle(P, calibrated(P, 12, stride=97), **opts)


def test_query_join():
    E = clusters(16600, 50, 10, 960)
    Q = np.concatenate([E[::5] + np.float32(0.01), clusters(2000, 50, 10, 970)])
    eps = calibrated(E, 15, stride=97)
    gi, gj = gpu_query_join(Q, E, eps)[:2]
    oi, oj = oracle.join(Q, E, eps)
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)
