"""GPU parity of the 16-bit filters' query-box kernel in workgroup units: one cell
holds every point, so that units of 256 queries are taken (asserted), cut at the
edges of parts and blocks; K padded to 16 and 32, few and many hits per tile, query
joins.  Pair lists must equal the oracle's.  And the planes that the box reads are
made only where it can be taken."""
import numpy as np
import pytest

import datagen
import oracle
from test_gpu_parity import assert_same_as_oracle, calibrated
from test_gpu_query import gpu_query_join

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ONE_CELL = dict(k=1, reorder=0)
WORKGROUP = 1  # sj_info.units


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def one_cell(kind, n, d, seed):
    """Points whose indexed dimension spans far less than any radius used here."""
    P = datagen.offgrid(kind, n, d, seed=seed)
    P[:, 0] *= np.float32(2.0 ** -12)
    return P


# a unit is 256 queries: two parts of 128 above 16 dimensions, the second of one
# query (385) and of none (1025, 1249: 225 in the last)
@pytest.mark.parametrize("n", [193, 224, 225, 255, 256, 385, 480, 1025, 1249])
@pytest.mark.parametrize("d", [2, 7, 8, 9, 16, 17, 24, 32])
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_edges(n, d, prec, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_BOX", "1")
    P = one_cell("uniform64", n, d, 900 + n + d)
    eps = calibrated(P, 12, stride=3)
    print("case box units", n, d, prec, flush=True)
    info = assert_same_as_oracle(P, eps, precision=prec, **ONE_CELL)
    assert info["units"] == WORKGROUP and info["n_cells"] == 1


@pytest.mark.parametrize("target", [2, 700])
@pytest.mark.parametrize("opts", [dict(), dict(min_batches=3), dict(sortidu=True)])
def test_selectivities_and_options(target, opts, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_BOX", "1")
    P = one_cell("mixture_f32", 4133, 16, 940)
    eps = calibrated(P, target, stride=5)
    print("case box units options", target, opts, flush=True)
    info = assert_same_as_oracle(P, eps, precision="fp16", **ONE_CELL, **opts)
    assert info["units"] == WORKGROUP


@pytest.mark.parametrize("m", [193, 225, 385])
def test_query_join(m, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_BOX", "1")
    E, Q = one_cell("uniform64", 1249, 20, 950), one_cell("uniform64", m, 20, 951)
    eps = calibrated(E, 12, stride=3)
    print("case box units query", m, flush=True)
    gi, gj, _, info, _ = gpu_query_join(Q, E, eps, precision="fp16", **ONE_CELL)
    assert info["units"] == WORKGROUP
    oi, oj = oracle.join(Q, E, eps)
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)


@pytest.mark.parametrize("d,made", [(24, True), (28, False)])
def test_planes_only_where_taken(d, made, monkeypatch):
    """32 bytes a point, above 24 dimensions only with the box forced."""
    from paper_1809_09930_amd import selfjoin as sj
    n = 1 << 20
    P = torch.rand((n, d), device="cuda")
    held = []
    for box in (None, None, "1"):  # (the first build makes what a process keeps)
        if box:
            monkeypatch.setenv("SJ_DEBUG_BOX", box)
        sj.selfjoin_release_cache()
        free = torch.cuda.mem_get_info()[0]
        h = sj.selfjoin_build_index(P, 0.3, precision="fp16", k=1)
        try:
            sj.selfjoin_release_cache()
            held.append(free - torch.cuda.mem_get_info()[0])
        finally:
            sj.selfjoin_free(h)
    extra = held[2] - held[1]
    assert abs(extra - (0 if made else 32 * n)) <= 4 << 20, held
