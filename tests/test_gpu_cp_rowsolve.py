"""CP-ALS's dense steps at the edges of their tiles: ranks around the powers of
two that the row solve and the elimination are laid out for, row counts around
the tiles of 64 to 256 rows and past one tile a workgroup.  After one sweep from
the same start: factors, column norms and Grams against the float64 oracle
(1e-4, the bar of the other one-sweep test: float32 sums through one solve), the
Grams against the stored factors themselves and unit columns (1e-6: float32
products summed in float64), the fit, and bitwise repeatability."""
import numpy as np
import pytest

import synth
from oracle import ref

from conftest import gpu_available
from gpu_util import f32, from_dev, rel_fro, tag

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("R,dims", [(1, [300, 20, 10]), (2, [129, 70, 9]), (3, [64, 65, 63]), (4, [257, 30, 20]),
                                    (5, [100, 90, 80]), (8, [65, 64, 200]), (15, [150, 127, 128]),
                                    (16, [90, 191, 66]), (17, [80, 193, 64]), (31, [200, 150, 100]),
                                    (32, [70000, 90, 65]), (33, [120, 40000, 64]), (48, [130, 110, 100]),
                                    (63, [128, 129, 127]), (64, [90, 100, 33000]), (8, [40, 30, 20, 50000])])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_sweep(R, dims, dtype):
    import torch
    import paper_1705_09905_amd as P
    t = synth.random_small(dims, 60000, seed=R)
    init = [f32(a) for a in synth.small_factors(dims, R, seed=R)]
    h = P.Tensor(t.idx, t.vals, dims)
    tag("rowsolve", R, dims, dtype)
    out, again = (P.cp_als(h, R, 1, init, dtype=dtype) for _ in range(2))
    for m in range(len(dims)):
        assert torch.equal(out["factors"][m], again["factors"][m])
        A, G = from_dev(out["factors"][m]), from_dev(out["grams"][m])
        assert rel_fro(G, A.T @ A) <= 1e-6
        norms = np.sqrt(np.diag(G))
        assert np.abs(norms[norms > 0] - 1).max() <= (1e-6 if dtype == "f32" else 2.0 ** -8)
    assert out["fits"] == again["fits"]
    if dtype == "f32":
        orc = ref.cp_als(dims, t.idx, f32(t.vals), R, init, 1, storage="f64")
        assert out["used_pinv"] == [0]
        for m in range(len(dims)):
            assert rel_fro(from_dev(out["factors"][m]), orc["factors"][m]) <= 1e-4
            assert rel_fro(from_dev(out["grams"][m]), orc["grams"][m]) <= 1e-4
        assert rel_fro(from_dev(out["lam"]), orc["lam"]) <= 1e-4
        assert abs(out["fits"][0] - orc["fits"][0]) <= 1e-4


@pytest.mark.parametrize("I", [1, 255, 256, 257, 131072, 131073, 300000])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gram_rows(I, dtype):
    import torch
    import paper_1705_09905_amd as P
    A = torch.randn(I, 33, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    t = P.Tensor([np.zeros(1, np.int32), np.zeros(1, np.int32)], [1.0], [I, 3])
    tag("gram-rows", I, dtype)
    G, D = t.gram(0, A), A.double()
    assert rel_fro(from_dev(G), from_dev(D.T @ D)) <= 1e-6
