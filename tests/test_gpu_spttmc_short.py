"""GPU parity of SpTTMc where rows have a few nonzeros each (a head in every other
step of four nonzeros), at the nonzero counts where its tiles change, and with the
last factor's columns held two and four a lane, on integer data (exact whatever the
order of the sums: every partial sum is an integer below 2^24)."""
import numpy as np
import pytest

import synth
from oracle import ref

from conftest import gpu_available
from gpu_util import from_dev, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _run(dims, Z, ranks, dtype, **build):
    from paper_1705_09905_amd import Tensor
    t = synth.random_small(dims, Z, seed=sum(ranks), value_kind="int")
    g = np.random.default_rng(sum(ranks))
    F = [g.integers(-3, 4, size=(d, r)).astype(np.float64) for d, r in zip(dims, ranks)]
    tag("ttmc-short", dims, Z, ranks, dtype, build)
    h = Tensor(t.idx, t.vals, dims).build(0, "mttkrp", **build)
    Y = from_dev(h.spttmc(0, [None] + [to_dev(f, dtype) for f in F[1:]]))
    np.testing.assert_array_equal(Y, ref.ttmc_coo(dims, t.idx, t.vals, F, 0))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("RA,RB", [(1, 18), (2, 32), (5, 40), (16, 36), (3, 64), (4, 132), (17, 32), (20, 34), (33, 62)])
def test_columns_per_lane(RA, RB, dtype):
    _run([1500, 40, 30], 4001, [1, RA, RB], dtype)
    _run([1500, 40, 30, 3], 2003, [1, 2, RA, RB], dtype)


@pytest.mark.parametrize("Z", [149999, 150000, 699999, 700001])
def test_tile_sizes(Z):
    _run([200000, 300, 200], Z, [1, 3, 5], "f32")
    _run([200000, 300, 200], Z, [1, 3, 5], "f32", xcd_blocks=8)
