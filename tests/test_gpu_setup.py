"""What a layer's set-up finds out about its lists, on layers wide enough that a workgroup of it takes several parts."""

import math

import numpy as np
import pytest

from tests import parity
from workloads import Layer, Problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("longest", [5, 262143, 262144, 299999])
def test_longest_row_anywhere_in_a_wide_layer(longest):
    """One fan-out row of 1500 entries among rows of one, at the first and last places a workgroup looks at: the
    small-sample product, which takes samples by the longest row, must not take the one that holds it."""
    import torch  # noqa: F401  (its HIP runtime is the one the library uses)

    import paper_1708_02937_amd as sd

    n, batch = 300000, 40
    rng = np.random.default_rng(longest)
    counts = np.ones(n, np.int64)
    counts[longest] = 1500
    row_ptr = np.zeros(n + 1, np.int64)
    np.cumsum(counts, out=row_ptr[1:])
    col = rng.integers(0, n, size=row_ptr[-1]).astype(np.int32)
    col[row_ptr[longest]:row_ptr[longest + 1]] = np.sort(rng.choice(n, 1500, replace=False))
    val = rng.uniform(0.5, 1, size=len(col)).astype(np.float32)
    layer = Layer(row_ptr, col, val, np.full(n, -0.1, np.float32))
    rows = [np.unique(np.append(rng.integers(0, n, size=20), [longest] if r % 2 else [])).astype(np.int32) for r in range(batch)]
    y_ptr = np.zeros(batch + 1, np.int64)
    np.cumsum([len(r) for r in rows], out=y_ptr[1:])
    y = (y_ptr, np.concatenate(rows), rng.uniform(0.5, 1, size=y_ptr[-1]).astype(np.float32))
    p = Problem(f"longest-{longest}", n, 1, batch, math.inf, [layer], y0_csr=y)
    net = sd.net_from_problem(p)
    print("[case] longest row", longest, flush=True)
    got = tuple(x.cpu().numpy() for x in net.forward_csr(*y))
    net.free()
    parity.compare(p, got)
