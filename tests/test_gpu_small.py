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
