"""An index of more than 2^26 cells with 27 neighbours each: a wave per list and
a wave per cell's work unit would each pass the 2^32 work-items of a dispatch."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_lattice_of_2_26_cells():
    from paper_1809_09930_amd import selfjoin as sj
    side, h = 407, 2.0 ** -9  # 67.4M lattice points, each alone in its cell
    x = torch.arange(side, device="cuda", dtype=torch.float32) * h
    P = torch.stack(torch.meshgrid(x, x, x, indexing="ij"), dim=-1).reshape(-1, 3).contiguous()
    n = side ** 3
    assert n > 2 ** 26
    print("case many cells", n, flush=True)
    handle = sj.selfjoin_build_index(P, 0.9995 * h, k=3)
    try:
        info = sj.selfjoin_get_info(handle)
        assert info["n_cells"] == n and info["candidates"] >= 16 * n
        assert sj.selfjoin_run(handle) == n  # points h apart: only the self pairs
        i = torch.empty(n, dtype=torch.int32, device="cuda")
        j = torch.empty(n, dtype=torch.int32, device="cuda")
        sj.selfjoin_fetch_pairs(handle, 0, i, j, max_pairs=n)
        every = torch.arange(n, dtype=torch.int32, device="cuda")
        assert torch.equal(i, every) and torch.equal(j, every)
    finally:
        sj.selfjoin_free(handle)
