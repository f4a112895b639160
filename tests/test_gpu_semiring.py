"""Semiring products: the LDS-resident form (dense input, at most 5119 neurons) and the row-wise form (CSR input),
at the edges of their slices, runs, windows and lane groups."""

import math

import numpy as np
import pytest

from tests.test_gpu_parity import SEMIRINGS, _mixed_length_layer
from workloads import Problem, tiny_random

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", SEMIRINGS)
@pytest.mark.parametrize("n,batch,lengths", [(1, 1, [1]), (65, 3, [0, 1, 4, 5]), (1025, 300, [3, 40, 0, 8]),
                                             (2048, 64, [33, 500]), (5119, 1030, [16, 2, 0]), (5120, 20, [16, 2, 0])])
def test_dense_input(name, n, batch, lengths):
    import oracle
    import torch

    import paper_1708_02937_amd as sd

    rng = np.random.default_rng(n)
    layer = _mixed_length_layer(rng, n, lengths)
    layer.val[rng.random(len(layer.val)) < 0.1] = 0.0
    y = rng.standard_normal((batch, n)).astype(np.float32)
    y[rng.random((batch, n)) < 0.3] = 0.0
    print("[case] semiring dense", name, n, batch, flush=True)
    net = sd.net_from_problem(Problem("s", n, 1, batch, math.inf, [layer], y0_dense=y))
    yd = torch.from_numpy(y).cuda()
    got = net.mxm(0, oracle.SEMIRINGS[name], yd).cpu().numpy()
    net.mxm(0, oracle.SEMIRINGS[name], yd, out=yd)  # in place
    net.free()
    assert got.tobytes() == oracle.mxm(name, n, layer, y).tobytes()
    assert yd.cpu().numpy().tobytes() == got.tobytes()


FOLD = {"max_plus": (lambda y, w: y + w, lambda a, b: a if a > b else b, -math.inf),
        "max_min": (lambda y, w: y if y < w else w, lambda a, b: a if a > b else b, -math.inf),
        "min_max": (lambda y, w: y if y > w else w, lambda a, b: a if a < b else b, math.inf)}


@pytest.mark.parametrize("name", sorted(FOLD))
def test_dense_input_non_finite(name):
    """A NaN is kept by the entry that brings it and dropped by the next, infinities select as numbers do: the
    reduction in ascending input order, entry by entry, with lists of every length around a block of four."""
    import oracle
    import torch

    import paper_1708_02937_amd as sd

    rng = np.random.default_rng(3)
    n, batch = 130, 5
    layer = _mixed_length_layer(rng, n, [0, 1, 2, 3, 4, 5, 6, 7, 8, 9])
    y = rng.standard_normal((batch, n)).astype(np.float32)
    for v in (math.nan, math.inf, -math.inf):
        y[rng.random((batch, n)) < 0.2] = v
    mul, add, zero = FOLD[name]
    want = np.full((batch, n), zero)
    for i, j, w in layer.entries():  # inputs ascending
        for r in range(batch):
            want[r, j] = add(want[r, j], mul(float(y[r, i]), w))
    net = sd.net_from_problem(Problem("s", n, 1, batch, math.inf, [layer], y0_dense=y))
    got = net.mxm(0, oracle.SEMIRINGS[name], torch.from_numpy(y).cuda()).cpu().numpy()
    net.free()
    assert np.array_equal(got, want.astype(np.float32), equal_nan=True)
    assert np.isnan(got).any() == (name == "max_plus")  # min and max of a NaN and a weight give the weight


@pytest.mark.parametrize("name", ["plus_times", "min_max", "xor_and"])
@pytest.mark.parametrize("n,batch,wd,yd", [(300, 40, 0.004, 0.3), (1000, 33, 0.0035, 0.5), (8192, 5, 0.001, 0.05),
                                           (8200, 4, 0.004, 0.1), (16384, 3, 0.004, 0.02), (16385, 3, 0.002, 0.03),
                                           (33000, 3, 0.0002, 0.02), (700, 70, 0.6, 0.2)])
def test_csr_input(name, n, batch, wd, yd):
    """Mean row lengths from 1 to 400 (every group width), one to three windows, both workgroup sizes; integer
    values, so every semiring is exact in any order."""
    import oracle

    import paper_1708_02937_amd as sd

    p = tiny_random(n, n, 1, batch, w_density=wd, y_density=yd, integer=True)
    rp, c, v = p.y0_csr
    yd_ = np.full((batch, n), {"min_max": math.inf}.get(name, 0.0), np.float32)
    yd_[np.repeat(np.arange(batch), np.diff(rp)), c] = v
    print("[case] semiring csr", name, n, batch, flush=True)
    net = sd.net_from_problem(p)
    got = net.mxm_csr(0, oracle.SEMIRINGS[name], rp, c, v).cpu().numpy()
    net.free()
    assert got.tobytes() == oracle.mxm(name, n, p.layers[0], yd_).tobytes()
