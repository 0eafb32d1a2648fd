"""FP32 joins that have to run on the matrix cores (asserted): result batches,
sortidu, partners within rounding of eps, ties, undersized buffers and query sets,
with their tiles' leading products first and with all products at once.  Up to 16
dimensions the form alone does not tell them from the vector norm form.  Pair lists
must equal the oracle's."""
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


@pytest.fixture(params=["0", "1"], autouse=True)
def lead(request, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_LEAD", request.param)
    return request.param


def matrix(info):
    return info["fp32_matrix"] == 1 and info["fp32_form"] == 2


@pytest.mark.parametrize("d", [10, 20, 40])
@pytest.mark.parametrize("opts", [dict(), dict(min_batches=3), dict(sortidu=True),
                                  dict(batch_pairs=40000)])
def test_options(d, opts, lead):
    P = datagen.offgrid("uniform64", 4700, d, seed=1100 + d)
    eps = calibrated(P, 15, stride=9)
    print("case route options", d, opts, lead, flush=True)
    assert matrix(assert_same_as_oracle(P, eps, k=1, **opts))


@pytest.mark.parametrize("d", [6, 16, 24, 30, 70])
def test_partners_at_radius(d, lead):
    base = datagen.offgrid("normal_binades", 4400, d, seed=1120 + d)
    base[:, 0] *= np.float32(2.0 ** -12)  # the indexed dimension: few cells
    eps = calibrated(base, 8, stride=9)
    P = np.concatenate([base, datagen.partners_near_radius(base, eps, 900, seed=1130 + d)])
    print("case route partners", d, lead, flush=True)
    info = assert_same_as_oracle(P, eps, k=1, reorder=0)
    assert matrix(info) and info["rechecks"] > 0


def test_undersized_buffers(lead, monkeypatch):
    monkeypatch.setenv("SJ_DEBUG_UNDERSIZE", "1")
    P = datagen.uniform_grid(4500, 12, 1140)
    eps = calibrated(P, 25, stride=9)
    for opts in (dict(), dict(min_batches=3)):
        assert matrix(assert_same_as_oracle(P, eps, k=1, **opts))


@pytest.mark.parametrize("m,d,runs", [(4300, 12, 1), (4100, 50, 1), (7, 12, 0)])
def test_query_join(m, d, runs, lead):
    """Seven queries stay on the vector ALUs, in difference form."""
    E = datagen.offgrid("uniform64", 4600, d, seed=1150 + d)
    Q = datagen.offgrid("uniform64", m, d, seed=1151 + d)
    Q[: m // 5] += np.float32(0.4)
    eps = calibrated(E, 15, stride=9)
    print("case route query", m, d, lead, flush=True)
    gi, gj, gd, info, _ = gpu_query_join(Q, E, eps, k=1)
    assert (info["fp32_matrix"], info["fp32_form"]) == (runs, 2 if runs else 1)
    oi, oj, os_ = oracle.join(Q, E, eps, with_dist=True)
    assert np.array_equal(gi, oi) and np.array_equal(gj, oj)
    np.testing.assert_allclose(gd, np.sqrt(os_), rtol=1e-5, atol=1e-30)


@pytest.mark.parametrize("form", [1, 2])
def test_vector_forms_say_so(form, lead):
    P = datagen.offgrid("uniform64", 4700, 10, seed=1160)
    info = assert_same_as_oracle(P, calibrated(P, 15, stride=9), k=1, fp32_form=form)
    assert (info["fp32_matrix"], info["fp32_form"]) == (0, form)


def test_little_memory_keeps_the_vector_form(lead):
    """The split rows are taken only where they fit a share of the free memory."""
    from paper_1809_09930_amd import selfjoin as sj
    n, d = 3_500_000, 16  # 0.49 GB of split rows
    P = torch.rand((n, d), device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    routes, pairs = [], []
    for leave in (None, 2 << 30):
        torch.cuda.empty_cache()
        sj.selfjoin_release_cache()
        held = []
        for part in (2 << 30, 64 << 20, 4 << 20):  # (one block of it all leaves more)
            while leave and torch.cuda.mem_get_info()[0] - part >= leave:
                held.append(torch.empty(part, dtype=torch.uint8, device="cuda"))
        assert not leave or torch.cuda.mem_get_info()[0] < leave + (64 << 20)
        print("case route memory", leave, lead, flush=True)
        h = sj.selfjoin_build_index(P, 0.1, k=4)
        try:
            routes.append(sj.selfjoin_get_info(h)["fp32_matrix"])
            total = sj.selfjoin_run(h)
            i, j = (torch.empty(total, dtype=torch.int32) for _ in range(2))
            sj.selfjoin_fetch_pairs(h, 0, i, j, max_pairs=total)
            pairs.append((i, j))
        finally:
            sj.selfjoin_free(h)
            del held
            torch.cuda.empty_cache()
    assert routes == [1, 0]
    assert torch.equal(pairs[0][0], pairs[1][0]) and torch.equal(pairs[0][1], pairs[1][1])
