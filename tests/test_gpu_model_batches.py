"""GPU parity of the model at the nonzeros where a lane group takes one batch of
nonzeros, several or as many as its lanes, and at order 5, on integer data (exact
whatever the order of the sums: every partial sum is an integer below 2^24)."""
import numpy as np
import pytest

from oracle import cpu

from conftest import gpu_available
from gpu_util import from_dev, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims,Z,R", [([300, 200, 100], 140001, 64), ([300, 200, 100], 270007, 33),
                                      ([300, 200, 100], 1100003, 50), ([300, 200, 100], 1100003, 10),
                                      ([300, 200, 100], 1100003, 130), ([90, 80], 560001, 20),
                                      ([40, 30, 20, 10, 9], 131, 7), ([40, 30, 20, 10, 9], 300001, 100)])
def test_batches(dims, Z, R, dtype):
    import torch
    from paper_1705_09905_amd import Tensor
    g = np.random.default_rng(R)
    idx = [g.integers(0, d, Z).astype(np.int32) for d in dims]
    F = [g.integers(-2, 3, (d, R)).astype(np.float64) for d in dims]
    h = Tensor(idx, np.ones(Z, np.float32), dims)
    tag("model-batches", dims, Z, R, dtype)
    out = torch.full((Z + 1,), float("nan"), device="cuda")
    got = h.model_at_nnz([to_dev(f, dtype) for f in F], out=out[:-1])
    np.testing.assert_array_equal(from_dev(got), cpu.model_at(idx, F))
    assert torch.isnan(out[-1])
