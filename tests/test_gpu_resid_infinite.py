"""The fused residual at ranks that the lanes' vectors do not divide, where the last
two lanes of a row hold some columns twice: an infinite element of a factor in such
a column gives what the definition gives (infinities, no NaN), elsewhere the rows
keep their values (1e-5, the bar of the other float32 comparisons: the oracle has
the factors as they are stored)."""
import numpy as np
import pytest

import synth

from conftest import gpu_available
from gpu_util import bf16, f32, from_dev, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("dtype,R,col", [("f32", 5, 1), ("f32", 10, 6), ("f32", 10, 7), ("f32", 63, 59), ("f32", 3, 1),
                                         ("bf16", 12, 5), ("bf16", 20, 15), ("bf16", 9, 1), ("bf16", 6, 2),
                                         ("f32", 8, 5), ("bf16", 16, 9)])
def test_infinite_column(dtype, R, col):
    import torch
    import paper_1705_09905_amd as P
    dims = [40, 30, 20]
    t = synth.random_small(dims, 3000, seed=R)
    A = [(bf16 if dtype == "bf16" else f32)(np.abs(a) + 0.5) for a in synth.small_factors(dims, R, seed=R)]
    A[1][7, col] = np.inf
    v = f32(t.vals)
    i = [np.asarray(x) for x in t.idx]
    hit = i[1] == 7
    assert 0 < hit.sum() < len(v) / 4
    d = (A[0][i[0]] * A[1][i[1]] * A[2][i[2]]).sum(1) - v
    G = np.zeros((dims[0], R))
    np.add.at(G, i[0], (d / len(v))[:, None] * A[1][i[1]] * A[2][i[2]])
    h = P.Tensor(t.idx, t.vals, dims)
    h.build(0, "mttkrp")
    tag("resid-inf", dtype, R, col)
    loss = torch.zeros((), dtype=torch.float64, device="cuda")
    got = from_dev(h.resid_spmttkrp(0, [to_dev(a, dtype) for a in A], loss=loss))
    assert np.isposinf(loss.item())
    assert np.isposinf(G).any() and np.isfinite(G).any()
    assert np.array_equal(np.isposinf(got), np.isposinf(G)) and not np.isnan(got).any()
    ok = np.isfinite(G)
    assert np.abs(got[ok] - G[ok]).max() <= 1e-5 * np.abs(G[ok]).max()
