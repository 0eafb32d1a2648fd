"""Device memory of FP32 matrix-core joins above 16 dimensions in result batches:
their filter accepts no pair itself, and the list of the pairs it leaves to FP64
has to be sized by a batch, not by the whole result.  Pair lists must equal the
oracle's."""
import numpy as np
import pytest

import datagen
import oracle
from test_gpu_parity import assert_same_as_oracle, calibrated

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_list_is_sized_by_a_batch():
    """A one-way run of 18M pairs in batches of 0.2M.  With the three result slots,
    the least list and the sampled count's, it takes some 60 MB; a list of the whole
    result alone would take 10 bytes per pair."""
    from paper_1809_09930_amd import selfjoin as sj
    E = datagen.offgrid("uniform64", 6000, 40, seed=860)
    eps = calibrated(E, 3000, stride=50)
    oi, oj = oracle.join(E, E, eps)
    tE = torch.from_numpy(E).cuda()
    he = sj.selfjoin_build_index(tE, eps, batch_pairs=200_000, mem_budget=32 << 20)
    hq = sj.selfjoin_build_query(he, tE)
    try:
        sj.selfjoin_release_cache()
        print("case list memory", len(oi), flush=True)
        free = torch.cuda.mem_get_info()[0]
        total = sj.selfjoin_run(hq)
        held = free - torch.cuda.mem_get_info()[0]  # the run's blocks, cached or kept
        info = sj.selfjoin_get_info(hq)
        assert info["fp32_form"] == 2 and info["batches"] >= 80
        assert total == len(oi) > 15_000_000
        i, j = (torch.empty(total, dtype=torch.int32) for _ in range(2))
        sj.selfjoin_fetch_pairs(hq, 0, i, j, max_pairs=total)
        assert np.array_equal(i.numpy(), oi) and np.array_equal(j.numpy(), oj)
        assert held < 8 * total, held
    finally:
        sj.selfjoin_free(hq)
        sj.selfjoin_free(he)


@pytest.mark.parametrize("mem_budget", [1 << 20, 40 << 20])
@pytest.mark.parametrize("d", [24, 40])
def test_small_budgets(d, mem_budget):
    """Few slots for the sampled count's list (it counts in parts then) and several
    batches that hand mirrored pairs on."""
    P = datagen.offgrid("uniform64", 4700, d, seed=870 + d)
    eps = calibrated(P, 700, stride=40)
    print("case list budget", d, mem_budget, flush=True)
    info = assert_same_as_oracle(P, eps, mem_budget=mem_budget)
    assert info["fp32_form"] == 2 and info["batches"] >= 2


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_wide_band_under_a_small_budget(prec):
    """Outliers widen the 16-bit band to most pairs: the sampled count's list does not
    hold them, and the batches still follow the pairs that are results."""
    P = datagen.offgrid("uniform64", 4500, 20, seed=880)
    eps = calibrated(P, 30, stride=9)
    P[:3] *= np.float32(2.0 ** 9)
    budget = 1 << 20
    print("case wide band", prec, flush=True)
    info = assert_same_as_oracle(P, eps, precision=prec, mem_budget=budget)
    assert info["rechecks"] > 10 * info["pairs"]
    assert info["batches"] <= 2 * info["pairs"] // (budget // 20) + 2
