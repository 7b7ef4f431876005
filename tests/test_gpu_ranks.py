"""GPU parity at ranks that the lanes' vector width (4 float32, 4 or 8
bfloat16 columns) does not divide: a row's last piece overlaps the one before,
rows shorter than a vector take narrower pieces, rank tiles end ragged.
Integer data is exact whatever the order of the sums (every partial sum is an
integer below 2^24), so a column written twice, skipped or counted twice in
the fused residual's dot product shows; factors and outputs also start at
addresses that are multiples of one element only."""
import numpy as np
import pytest

import synth
from oracle import cpu

from conftest import gpu_available
from gpu_util import TOL_F32, bf16, f32, from_dev, rel_fro, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DIMS = {2: [60, 40], 3: [40, 30, 20], 4: [20, 15, 10, 8], 5: [12, 10, 8, 6, 5]}


def _offset(x):
    """The same matrix one element past an allocation's start."""
    import torch
    buf = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)
    return buf[1:].view(x.shape).copy_(x)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("R", [1, 2, 3, 5, 6, 7, 9, 10, 13, 25, 31, 33, 50, 63, 65, 127, 130, 255])
def test_any_rank_exact(R, dtype):
    import torch
    from paper_1705_09905_amd import Tensor
    for order, dims in DIMS.items():
        t = synth.random_small(dims, 3001 if order > 2 else 1501, seed=R, value_kind="int")
        F = synth.small_factors(dims, R, seed=R, kind="int")
        dev = [_offset(to_dev(f, dtype)) for f in F]
        mode = R % order
        for lane_cols in ((0,) if dtype == "f32" else (0, 4, 8)):
            tag("rank", R, dtype, dims, "mode", mode, "lane_cols", lane_cols)
            h = Tensor(t.idx, t.vals, dims).build(mode, "mttkrp", tile_nnz=256, lane_cols=lane_cols)
            h.build(mode, "ttm", tile_nnz=256, lane_cols=lane_cols)
            out = _offset(torch.full((dims[mode], R), float("nan"), device="cuda"))
            np.testing.assert_array_equal(from_dev(h.spmttkrp(mode, dev, out=out)),
                                          cpu.mttkrp(dims, t.idx, t.vals, F, mode))
            Y = _offset(torch.full((h.info(mode, "ttm")["nseg"], R), float("nan"), device="cuda"))
            np.testing.assert_array_equal(from_dev(h.spttm(mode, dev[mode], out=Y)),
                                          cpu.ttm(dims, t.idx, t.vals, F[mode], mode)[1])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("R", [1, 2, 3, 5, 7, 9, 25, 33, 61, 63])
def test_any_rank_residual(R, dtype):
    import torch
    from paper_1705_09905_amd import Tensor
    for order, dims in DIMS.items():
        t = synth.random_small(dims, 3001 if order > 2 else 1501, seed=R)
        F = [f32(f) if dtype == "f32" else bf16(f) for f in synth.small_factors(dims, R, seed=R)]
        exp_loss, exp = cpu.mse_grad(dims, t.idx, f32(t.vals), F)
        mode = R % order
        loss = torch.zeros((), dtype=torch.float64, device="cuda")
        tag("rank-resid", R, dtype, dims, "mode", mode)
        h = Tensor(t.idx, t.vals, dims).build(mode, tile_nnz=256)
        G = from_dev(h.resid_spmttkrp(mode, [_offset(to_dev(f, dtype)) for f in F], loss=loss))
        assert rel_fro(G, exp[mode]) <= TOL_F32, rel_fro(G, exp[mode])
        assert abs(loss.item() - exp_loss) <= 1e-5 * exp_loss


def test_residual_rank_limits():
    from paper_1705_09905_amd import FcooError, Tensor
    t = synth.random_small([9, 8, 7], 100, seed=1)
    h = Tensor(t.idx, t.vals, t.dims).build(0)
    for dtype, R, ok in [("f32", 64, True), ("f32", 65, False), ("bf16", 65, False), ("bf16", 100, False),
                         ("bf16", 120, True), ("bf16", 128, True), ("bf16", 136, False)]:
        dev = [to_dev(f, dtype) for f in synth.small_factors(t.dims, R, seed=R)]
        if ok:
            h.resid_spmttkrp(0, dev)
        else:
            with pytest.raises(FcooError):
                h.resid_spmttkrp(0, dev)
