"""GPU parity of segments that cross work tiles: none, one, two and more tiles
wholly inside a segment, up to chains past the length that gets a workgroup of
its own, closed by a later segment or by the end of the tensor, at ranks
narrower and wider than the workgroup that finishes them.  Integer data is
exact whatever the order of the sums (every partial sum is an integer below
2^24), so a partial left out or counted twice shows."""
import numpy as np
import pytest

from oracle import cpu

from conftest import gpu_available
from gpu_util import from_dev, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TILE = 256
# nonzeros of each slice: they start at every phase of a tile
LENGTHS = [3, TILE, TILE + 1, 2 * TILE - 7, 1, 3 * TILE, 2, 4 * TILE + 5, 65 * TILE, 9, 66 * TILE + 3, 1, 1, 300]
MORE = [5] * 700 + [2 * TILE + 100]


def _tensor(lengths, rng):
    rows = np.repeat(np.arange(len(lengths)), lengths)
    n = len(rows)
    dims = [len(lengths), 150, 130]
    j = np.concatenate([np.arange(k) for k in lengths])                  # distinct coordinates within a slice
    idx = [rows.astype(np.int32), (j // 130 % 150).astype(np.int32), (j % 130).astype(np.int32)]
    return dims, idx, rng.integers(-2, 3, n).astype(np.float32)


@pytest.mark.parametrize("R", [1, 8, 16, 48, 100, 256])
@pytest.mark.parametrize("lengths", [LENGTHS, MORE, LENGTHS + MORE])
def test_chains_exact(lengths, R):
    from paper_1705_09905_amd import Tensor
    rng = np.random.default_rng(R)
    dims, idx, vals = _tensor(lengths, rng)
    F = [rng.integers(-2, 3, (d, R)).astype(np.float64) for d in dims]
    for dtype in ("f32", "bf16"):
        dev = [to_dev(f, dtype) for f in F]
        for device in (False, True):
            tag("chains", R, dtype, len(lengths), "device build", device)
            h = Tensor(idx, vals, dims).build(0, "mttkrp", tile_nnz=TILE, device=device)
            np.testing.assert_array_equal(from_dev(h.spmttkrp(0, dev)), cpu.mttkrp(dims, idx, vals, F, 0))


def test_chains_wide_rows():
    from paper_1705_09905_amd import Tensor
    rng = np.random.default_rng(7)
    dims, idx, vals = _tensor(LENGTHS, rng)
    F = [rng.integers(-2, 3, (d, r)).astype(np.float64) for d, r in zip(dims, (1, 40, 36))]
    h = Tensor(idx, vals, dims).build(0, "mttkrp", tile_nnz=TILE)
    exp = np.zeros((dims[0], 40 * 36))
    np.add.at(exp, idx[0], vals[:, None] * (F[1][idx[1]][:, :, None] * F[2][idx[2]][:, None, :]).reshape(-1, 40 * 36))
    np.testing.assert_array_equal(from_dev(h.spttmc(0, [to_dev(f, "f32") for f in F])), exp)
