"""GPU parity of candidate runs and work units built with several lanes per
list: neighbour lists of a few cells (8 lanes), of tens and of hundreds of cells
with gaps (a wave, several steps), for the symmetric join, result batches, the
per-block ranges of sortidu and query joins.  Pair lists must equal the oracle's."""
import numpy as np
import pytest

import datagen
import oracle
from test_gpu_parity import assert_same_as_oracle
from test_gpu_query import gpu_query_join

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# d, cells along a dimension: lists of 1, up to 3, 9, 27, 81 and 729 cells
LISTS = [(2, 1, 1), (1, 1, 40), (2, 2, 12), (3, 3, 7), (4, 4, 5), (6, 6, 3)]


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def points(n, d, seed):
    # thin out a corner, so that lists have gaps and cells differ in size
    P = datagen.offgrid("uniform64", n, d, seed=seed)
    span = P.max(axis=0) - P.min(axis=0)
    far = (P > P.min(axis=0) + 0.6 * span).sum(axis=1) >= max(1, d // 2)
    keep = ~far | (np.arange(n) % 9 == 0)
    return np.ascontiguousarray(P[keep])


@pytest.mark.parametrize("opts", [dict(), dict(batch_pairs=4000), dict(sortidu=True),
                                  dict(precision="fp16")])
@pytest.mark.parametrize("d,k,cells", LISTS)
def test_self_join(d, k, cells, opts):
    P = points(2600, d, 700 + d)
    eps = float((P.max(axis=0) - P.min(axis=0)).max()) / cells
    eps *= 0.1 if d == 2 and k == 1 else 0.999
    print("case runs", d, k, cells, opts, flush=True)
    assert_same_as_oracle(P, eps, k=k, **opts)


@pytest.mark.parametrize("d,k,cells", LISTS[2:])
def test_query_join(d, k, cells):
    E = points(2000, d, 720 + d)
    Q = points(900, d, 730 + d)
    Q[:100] += np.float32(0.4)
    eps = float((E.max(axis=0) - E.min(axis=0)).max()) / cells * 0.999
    gi, gj = gpu_query_join(Q, E, eps, k=k)[:2]
    oi, oj = oracle.join(Q, E, eps)
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)
