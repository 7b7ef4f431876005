"""Builds on the GPU take their memory from a pool: repeated builds, builds of
several sizes and layouts in turn, of several handles and from several threads
stay bit-exact with the host builder, and operations queued before a rebuild
read the arrays that they were launched on."""
import threading

import numpy as np
import pytest

import synth

from conftest import gpu_available
from gpu_util import from_dev, tag, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _same(h, d, mode, op):
    a, b = h.export(mode, op), d.export(mode, op)
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


def _cycle(dims, Z, seed, rounds):
    from paper_1705_09905_amd import Tensor
    t = synth.random_small(dims, Z, seed=seed, value_kind="int")
    host, dev = Tensor(t.idx, t.vals, dims), Tensor(t.idx, t.vals, dims)
    for k in range(rounds):
        for mode in range(len(dims)):
            for op, xcd in (("mttkrp", 0), ("ttm", 0), ("mttkrp", 8)):
                host.build(mode, op, host_only=True, xcd_blocks=xcd)
                dev.build(mode, op, device=True, xcd_blocks=xcd)
                _same(host, dev, mode, op)


@pytest.mark.parametrize("dims,Z", [([50, 40, 30], 20000), ([9, 8, 7, 6, 5], 9000), ([1, 3, 70000], 5000)])
def test_repeated_builds(dims, Z):
    tag("pool", dims, Z)
    _cycle(dims, Z, Z, 3)


def test_threads():
    tag("pool-threads")
    errors = []

    def work(k):
        try:
            _cycle([40 + k, 30, 20], 3000 + 777 * k, k, 2)
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for x in ts:
        x.start()
    for x in ts:
        x.join()
    assert not errors, errors


def test_rebuild_behind_queued_work():
    import torch
    from paper_1705_09905_amd import Tensor
    t = synth.random_small([300, 200, 100], 200000, seed=3, value_kind="int")
    F = [to_dev(f) for f in synth.small_factors(t.dims, 16, seed=3, kind="int")]
    h, other = (Tensor(t.idx, t.vals, t.dims).build(0, device=True) for _ in range(2))
    want = from_dev(h.spmttkrp(0, F))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    tag("pool-queued")
    outs = []
    for k in range(5):
        with torch.cuda.stream(side):
            outs += [h.spmttkrp(0, F) for _ in range(20)]
        h.build(0, device=True, xcd_blocks=8 * (k % 2))      # on the other stream, same handle
        other.build(k % 3, "ttm", device=True)
    torch.cuda.synchronize()
    for o in outs:
        np.testing.assert_array_equal(from_dev(o), want)
