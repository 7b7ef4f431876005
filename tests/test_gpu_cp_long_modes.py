"""CP-ALS from a fresh handle where a smaller mode's Gram takes more workgroups
than the largest mode's (float32 past 131,072 rows, bfloat16 past 524,288): one
sweep against the float64 oracle (1e-4, the bar of the other one-sweep tests),
the Grams against the stored factors (1e-6: products exact in float32 or better,
summed in float64 past 256 rows), bitwise repeatability."""
import pytest

import synth
from oracle import ref

from conftest import gpu_available
from gpu_util import f32, from_dev, rel_fro, tag

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("dtype,R,dims", [("f32", 8, [140000, 120000, 50]), ("f32", 33, [131073, 131072, 50]),
                                          ("bf16", 8, [600000, 500000, 50]), ("bf16", 33, [524289, 524288, 50]),
                                          # (rows past one workgroup's first tiles, for every row length)
                                          ("f32", 1, [70000, 65537, 9]), ("f32", 2, [140001, 300, 9]),
                                          ("f32", 4, [66000, 300, 50]), ("f32", 16, [132000, 300, 50]),
                                          ("bf16", 1, [262144, 300, 9]), ("bf16", 3, [262145, 70000, 50]),
                                          ("bf16", 7, [200000, 300, 50]), ("bf16", 20, [262145, 66000, 50])])
def test_fresh_sweep(dtype, R, dims):
    import torch
    import paper_1705_09905_amd as P
    t = synth.random_small(dims, 60000, seed=R)
    init = [f32(a) for a in synth.small_factors(dims, R, seed=R)]
    tag("long-modes", dtype, R, dims)
    out, again = (P.cp_als(P.Tensor(t.idx, t.vals, dims), R, 1, init, dtype=dtype) for _ in range(2))
    assert out["fits"] == again["fits"] and torch.equal(out["lam"], again["lam"])
    for m in range(3):
        assert torch.equal(out["factors"][m], again["factors"][m])
        A = from_dev(out["factors"][m])
        assert rel_fro(from_dev(out["grams"][m]), A.T @ A) <= 1e-6
    if dtype == "f32":
        orc = ref.cp_als(dims, t.idx, f32(t.vals), R, init, 1, storage="f64")
        for m in range(3):
            assert rel_fro(from_dev(out["factors"][m]), orc["factors"][m]) <= 1e-4
        assert rel_fro(from_dev(out["lam"]), orc["lam"]) <= 1e-4
        assert abs(out["fits"][0] - orc["fits"][0]) <= 1e-4
