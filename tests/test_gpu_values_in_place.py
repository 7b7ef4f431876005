"""SpMTTKRP with replaced values that lie in the result's own memory: the result is
that of values of their own (bit for bit: the same sums)."""
import pytest

import synth

from conftest import gpu_available
from gpu_util import f32, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("opts", [{}, {"single_pass": True}, {"xcd_blocks": 8}])
@pytest.mark.parametrize("offset", [0, 1001])
def test_in_place(opts, offset):
    import torch
    import paper_1705_09905_amd as P
    dims, R, Z = [500, 300, 200], 16, 4000
    t = synth.random_small(dims, Z, seed=3)
    h = P.Tensor(t.idx, t.vals, dims)
    h.build(0, "mttkrp", **opts)
    F = [to_dev(f32(a)) for a in synth.small_factors(dims, R, seed=3)]
    buf = torch.randn(dims[0] * R, device="cuda")
    g = buf[offset:offset + Z]
    want = h.spmttkrp_values(0, g.clone(), F)
    tag("values-in-place", opts, offset)
    got = h.spmttkrp_values(0, g, F, out=buf.view(dims[0], R))
    assert torch.equal(got, want)
