"""GPU parity of the model at the nonzeros and of SpMTTKRP with replaced values,
at ranks the lanes' vector width does and does not divide, one and several rank
tiles, orders 2 to 6, and nonzero counts around a wave's 64 and a workgroup's
256.  Integer data is exact whatever the order of the sums (every partial sum is
an integer below 2^24), so a column summed twice, or a value of another nonzero,
shows."""
import numpy as np
import pytest

import synth
from oracle import cpu

from conftest import gpu_available
from gpu_util import from_dev, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DIMS = {2: [60, 40], 3: [40, 30, 20], 4: [20, 15, 10, 8], 6: [9, 8, 7, 6, 5, 4]}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("R", [1, 2, 3, 4, 6, 8, 9, 16, 25, 33, 64, 100, 130, 256])
def test_model_exact(R, dtype):
    import torch
    from paper_1705_09905_amd import Tensor
    for order, dims in DIMS.items():
        for nnz in (1, 63, 65, 257, 1301):
            tag("model", R, dtype, dims, nnz)
            t = synth.random_small(dims, nnz, seed=R + nnz, value_kind="int")
            F = [np.clip(f, -2, 2) for f in synth.small_factors(dims, R, seed=R, kind="int")]
            exp = np.prod([f[i] for f, i in zip(F, t.idx)], axis=0).sum(axis=1)
            out = torch.full((len(t.vals) + 1,), float("nan"), device="cuda")
            h = Tensor(t.idx, t.vals, dims)
            got = h.model_at_nnz([to_dev(f, dtype) for f in F], out=out[:-1])
            np.testing.assert_array_equal(from_dev(got), exp)
            assert torch.isnan(out[-1])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("R", [1, 3, 4, 8, 16, 25, 64, 130])
def test_replaced_values_exact(R, dtype):
    from paper_1705_09905_amd import Tensor
    for order, dims in DIMS.items():
        for nnz, device, blocks in ((1, False, 0), (257, True, 0), (1301, False, 0), (1301, True, 0), (1301, True, 8)):
            if blocks and order == 2:
                continue
            tag("values", R, dtype, dims, nnz, device, blocks)
            t = synth.random_small(dims, nnz, seed=R + nnz, value_kind="int")
            F = [np.clip(f, -2, 2) for f in synth.small_factors(dims, R, seed=R, kind="int")]
            g = np.random.default_rng(nnz).integers(-3, 4, len(t.vals)).astype(np.float32)
            mode = R % order
            h = Tensor(t.idx, t.vals, dims).build(mode, "mttkrp", tile_nnz=256, device=device, xcd_blocks=blocks)
            got = h.spmttkrp_values(mode, to_dev(g, "f32"), [to_dev(f, dtype) for f in F])
            np.testing.assert_array_equal(from_dev(got), cpu.mttkrp(dims, t.idx, g, F, mode))
