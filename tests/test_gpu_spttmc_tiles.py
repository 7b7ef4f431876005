"""GPU parity of SpTTMc's matrix-core kernel at the edges of its 16 x 16 column
blocks, of its 64-nonzero chunks and of its tiles, on integer data (exact
whatever the order of the sums: every partial sum is an integer below 2^24),
for two to four product modes, both storage types, both layouts; rows of one
segment holding an infinity leave the others alone; a factor of more than
4 GiB."""
import numpy as np
import pytest

import synth
from oracle import ref

from conftest import gpu_available
from gpu_util import from_dev, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _run(t, ranks, mode, dtype, **build):
    from paper_1705_09905_amd import Tensor
    g = np.random.default_rng(sum(ranks))
    F = [g.integers(-3, 4, size=(d, r)).astype(np.float64) for d, r in zip(t.dims, ranks)]
    tag("ttmc", t.dims, t.nnz, ranks, "mode", mode, dtype, build)
    h = Tensor(t.idx, t.vals, t.dims).build(mode, "mttkrp", **build)
    Y = from_dev(h.spttmc(mode, [None if m == mode else to_dev(f, dtype) for m, f in enumerate(F)]))
    np.testing.assert_array_equal(Y, ref.ttmc_coo(t.dims, t.idx, t.vals, F, mode))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ranks", [[1, 1, 1], [15, 16, 17], [16, 17, 15], [17, 31, 33], [33, 16, 64], [64, 65, 1],
                                   [1, 5, 130], [8, 40, 40]])
def test_column_blocks(ranks, dtype):
    t = synth.random_small([40, 30, 20], 5003, seed=sum(ranks), value_kind="int")
    for mode in range(3):
        _run(t, ranks, mode, dtype)


@pytest.mark.parametrize("dims,ranks", [([30, 20], [7, 19]), ([12, 10, 8, 6], [3, 5, 4, 17]),
                                        ([9, 8, 7, 6, 5], [2, 3, 4, 5, 3]), ([5, 4, 4, 3, 3, 3], [2, 2, 3, 2, 3, 2])])
def test_product_mode_counts(dims, ranks):
    t = synth.random_small(dims, 550, seed=len(dims), value_kind="int")
    for mode in range(len(dims)):
        _run(t, ranks, mode, "f32")


@pytest.mark.parametrize("Z", [1, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1024, 1025, 4096, 4097, 9000])
@pytest.mark.parametrize("rows", [1, 3, 5000])
def test_chunk_and_tile_edges(Z, rows):
    t = synth.random_small([rows, 60, 50], Z, seed=Z, value_kind="int")
    _run(t, [1, 16, 5], 0, "f32")
    _run(t, [1, 16, 5], 0, "f32", tile_nnz=256)


@pytest.mark.parametrize("T", [256, 512, 1024, 4096])
def test_blocked_layout(T):
    t = synth.random_small([300, 200, 100], 60000, seed=T, value_kind="int")
    _run(t, [1, 16, 20], 0, "f32", tile_nnz=T, xcd_blocks=8)


def test_infinity_stays_in_its_rows():
    import torch
    from paper_1705_09905_amd import Tensor
    t = synth.random_small([500, 40, 30], 4000, seed=9)
    F = [to_dev(f) for f in synth.small_factors(t.dims, 16, seed=9)]
    h = Tensor(t.idx, t.vals, t.dims).build(0)
    clean = h.spttmc(0, F)
    F[1][7, 3] = float("inf")
    F[2][11, 5] = float("nan")
    tag("ttmc-inf")
    hit = torch.zeros(500, dtype=torch.bool, device="cuda")
    bad = (t.idx[1] == 7) | (t.idx[2] == 11)
    hit[torch.as_tensor(t.idx[0][bad].astype(np.int64), device="cuda")] = True
    Y = h.spttmc(0, F)
    assert bad.any() and not hit.all()
    assert torch.equal(Y[~hit], clean[~hit])
    assert not torch.isfinite(Y[hit]).all()


def test_factor_over_4_GiB():
    import torch
    from paper_1705_09905_amd import Tensor
    dims, Z = [50, 17_000_000, 9], 3000
    g = np.random.default_rng(4)
    idx = [g.integers(0, d, size=Z).astype(np.int32) for d in dims]
    idx[1][:2] = [0, dims[1] - 1]
    vals = g.integers(1, 5, size=Z).astype(np.float64)
    U = torch.zeros(dims[1], 64, device="cuda")
    rows = torch.as_tensor(idx[1].astype(np.int64), device="cuda")
    U[rows] = torch.as_tensor(g.integers(-3, 4, size=(Z, 64)).astype(np.float32), device="cuda")
    V = torch.as_tensor(g.integers(-3, 4, size=(dims[2], 5)).astype(np.float32), device="cuda")
    tag("ttmc-wide", dims)
    Y = from_dev(Tensor(idx, vals, dims).build(0).spttmc(0, [None, U, V]))
    u, v = from_dev(U[rows]), from_dev(V)[idx[2]]
    exp = np.zeros((dims[0], 64 * 5))
    np.add.at(exp, idx[0], vals[:, None] * (u[:, :, None] * v[:, None, :]).reshape(Z, -1))
    np.testing.assert_array_equal(Y, exp)
