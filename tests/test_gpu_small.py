"""GPU parity at the sizes where the short sorts and scans of one workgroup end:
point sets (sorted keys with ids) and results (keys alone) around a wave, a tile
and 4096 keys, and tables of one cell per point around the scans' tile sizes.
Pair lists must equal the oracle's."""
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


@pytest.mark.parametrize("opts", [dict(), dict(precision="fp16"), dict(sortidu=True)])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 1023, 1025, 2048, 4095, 4096, 4097])
def test_keys_and_results(n, opts):
    P = datagen.offgrid("uniform64", n, 3, seed=800 + n)
    print("case small", n, opts, flush=True)
    assert_same_as_oracle(P, calibrated(P, min(2, n / 8), stride=1) if n > 64 else 0.2, **opts)


@pytest.mark.parametrize("n", [2047, 2049, 8191, 8193, 16385, 32767, 32769])
def test_a_cell_per_point(n):
    # distinct multiples of 1 / 2^16, eps half of that: every point alone in its cell
    x = np.random.default_rng(n).permutation(1 << 16)[:n].astype(np.float32) / np.float32(1 << 16)
    print("case cells", n, flush=True)
    assert_same_as_oracle(np.ascontiguousarray(x[:, None]), 0.5 / (1 << 16), k=1)


@pytest.mark.parametrize("groups", ["0", "1"])
@pytest.mark.parametrize("n", [300, 1023, 1024, 1025, 5000])
def test_without_sampled_count(n, groups, monkeypatch):
    """All pairs of up to 1024 points fit the least result buffer (every pair is a
    result here), more go through the sampled count; units of single cells and of
    groups of them."""
    monkeypatch.setenv("SJ_DEBUG_GROUPS", groups)
    P = datagen.offgrid("uniform64", n, 4, seed=850 + n)
    print("case count", n, groups, flush=True)
    assert_same_as_oracle(P, 10.0 * float(np.ptp(P)) if n <= 1025 else calibrated(P, 9, stride=3))
    assert_same_as_oracle(P, calibrated(P, 5, stride=3), precision="bf16")
    assert_same_as_oracle(P, calibrated(P, 5, stride=3), mem_budget=1000)
