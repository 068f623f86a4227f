"""The fp32 tiles of 16 waves that serve N/M <= 1/16 above 128 rows, at the
edges of tiles and stages, against the oracle (exact on integers), and from the
debug build that poisons every LDS fill."""
import ctypes

import numpy as np
import pytest

import oracle
from nm_workloads import make_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2503_01253_amd as nm  # noqa: E402
from paper_2503_01253_amd.binding import load, tuning_string  # noqa: E402
from paper_2503_01253_amd.build import POISON_LIB_PATH  # noqa: E402

# (m, k, n, N, M, V): one to eight compressed rows a stage, a partial last
# stage, ragged rows and columns, blocks wider than a tile
SHAPES = [
    (129, 128, 512, 2, 32, 32), (255, 416, 544, 1, 32, 32), (140, 384, 288, 1, 16, 32), (300, 320, 1024, 3, 64, 64),
    (130, 640, 512, 8, 128, 512), (128, 256, 256, 1, 128, 128),
]


@pytest.mark.parametrize("poison", [False, True])
@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("tile", ["128x512m32q", "128x256m32q"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_exact(shape, tile, splits, poison):
    m, k, n, N, M, V = shape
    tuning = {"TILE": tile, "SPLITS": splits}
    assert f"<{tile},bv1,ka128," in nm.nmspmm_kernel_name(m, n, k, N, M, V, tuning=tuning)
    A, Bp, _ = make_inputs(m, k, n, N, M, V, m + k, "int")
    Bc, idx = oracle.compress(Bp, N, M, V)
    dA, dBc, didx = (torch.from_numpy(x).cuda() for x in (A, Bc, idx))
    C = torch.full((m, n), float("nan"), device="cuda")
    L = load(POISON_LIB_PATH) if poison else nm.lib()
    st = L.nmspmm_run_tuned(dA.data_ptr(), dBc.data_ptr(), didx.data_ptr(), C.data_ptr(), m, n, k, N, M, V,
                            ctypes.c_float(1.0), None, 0, None, 0, tuning_string(tuning),
                            torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert np.array_equal(C.cpu().numpy().astype(np.float64), oracle.spmm(A, Bc, idx, m, n, k, N, M, V))


@pytest.mark.parametrize("N", [1, 2])
def test_two_column_regions(N):
    """28 column tiles of 512 in one round, the other 5120 columns in a second."""
    m, k, n, M, V = 1152, 160, 19456, 32, 32
    name = nm.nmspmm_kernel_name(m, n, k, N, M, V)
    assert name.startswith("nm_tiled_kernel<128x512m32q,") and "+cols14336:nm_tiled_kernel<128x256m32q," in name
    A, Bp, _ = make_inputs(m, k, n, N, M, V, 3 + N, "int")
    Bc, idx = oracle.compress(Bp, N, M, V)
    C = torch.full((m, n), float("nan"), device="cuda")
    nm.nmspmm_run(*(torch.from_numpy(x).cuda() for x in (A, Bc, idx)), C, m, n, k, N, M, V)
    assert np.array_equal(C.cpu().numpy().astype(np.float64), oracle.spmm(A, Bc, idx, m, n, k, N, M, V))
