"""The vector packer of nmspmm_compress_device (M a power of two up to 32, V a
multiple of 4) at its edges, against the oracle byte for byte: windows that do
not fill a 32-row tile, blocks that do not fill 256 columns, every thread
layout, and arrays that are not 16-byte aligned (the other packers)."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2503_01253_amd as nm  # noqa: E402

# (k, n, N, M, V)
SHAPES = [
    (20, 4, 2, 4, 4), (36, 12, 1, 4, 4), (7, 260, 1, 1, 4), (34, 40, 1, 2, 8), (40, 1000, 3, 8, 8),
    (48, 288, 7, 16, 96), (96, 1024, 8, 32, 256), (64, 800, 32, 32, 200), (32, 2816, 8, 32, 32), (80, 528, 4, 16, 16),
]


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_byte_for_byte(shape, ties, offset):
    k, n, N, M, V = shape
    rng = np.random.default_rng(k * n + M)
    B = (rng.integers(-1, 2, (k, n)) if ties else rng.standard_normal((k, n))).astype(np.float32)
    w, q = k // M * N, n // V
    store = torch.empty(offset + k * n, device="cuda")
    dB = store[offset:].view(k, n)
    dB.copy_(torch.from_numpy(B))
    Bc, idx = torch.full((w, n), float("nan"), device="cuda"), torch.full((w, q), 255, dtype=torch.uint8, device="cuda")
    nm.nmspmm_compress_device(dB, Bc, idx, N, M, V)
    Bc_o, idx_o = oracle.compress(B, N, M, V)
    assert np.array_equal(idx.cpu().numpy(), idx_o)
    assert Bc.cpu().numpy().tobytes() == Bc_o.tobytes()
