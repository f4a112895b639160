"""The dense-Y forward with the activations of a few samples resident in LDS (layers of at most 5119 neurons).

With the profiling log on, a range of small layers runs on the neuron-major gather instead, which sums every
output in the same order, so the two results must be equal bit for bit; every case is also compared with the
oracle."""

import math

import numpy as np
import pytest

from tests import parity
from tests.test_gpu_parity import _mixed_length_layer
from workloads import Problem, dense_to_csr, make_config

pytestmark = pytest.mark.gpu

# n around the 64-neuron slices, the 1024-neuron runs and the largest width; batches around one, two and four
# samples per workgroup and past one round of workgroups; list lengths around the blocks of four entries
CASES = [(1, 1, 2, [1], 0), (63, 5, 3, [0, 1, 3, 4], 0), (64, 64, 2, [5, 8, 9], 1), (65, 255, 2, [16], 0),
         (1023, 257, 2, [0, 7, 12, 400], 0), (1024, 64, 33, [16, 2], 0), (1025, 513, 2, [4, 31], 1),
         (2047, 1030, 1, [33, 1, 0, 90], 0), (3000, 100, 2, [20, 700, 3], 0), (4096, 64, 1, [64, 50, 0], 1),
         (4095, 9, 3, [17, 18], 0), (5119, 255, 2, [32, 3, 48], 0), (5119, 3, 1, [2000, 1, 4], 0)]


def _problem(n, batch, L, lengths, seed):
    rng = np.random.default_rng(seed)
    layers = [_mixed_length_layer(rng, n, lengths[k % len(lengths):] + lengths[:k % len(lengths)])
              for k in range(min(L, 3))]
    y = rng.random((batch, n), dtype=np.float32)
    y[rng.random((batch, n)) < 0.3] = 0.0
    return Problem(f"resident-{n}-{batch}", n, L, batch, [math.inf, 2.5][seed % 2],
                   [layers[k % len(layers)] for k in range(L)], y0_dense=y)


@pytest.mark.parametrize("n,batch,L,lengths,bias_mode", CASES)
def test_resident_forward(n, batch, L, lengths, bias_mode):
    import torch

    import paper_1708_02937_amd as sd

    p = _problem(n, batch, L, lengths, n + batch)
    print("[case] resident", n, batch, L, bias_mode, flush=True)
    net = sd.net_from_problem(p, bias_mode=bias_mode)
    y = torch.from_numpy(p.y0_dense).cuda()
    got = net.forward_dense(y).cpu().numpy()
    net.set_profiling(True)
    layerwise = net.forward_dense(y).cpu().numpy()
    net.set_profiling(False)
    assert got.tobytes() == layerwise.tobytes()
    if L > 1:  # in place, and in two ranges
        z = y.clone()
        net.forward_dense(z, out=z)
        assert z.cpu().numpy().tobytes() == got.tobytes()
        two = net.forward_dense(net.forward_dense(y, k0=0, k1=1), k0=1, k1=L)
        assert two.cpu().numpy().tobytes() == got.tobytes()
    net.free()
    parity.compare(p, dense_to_csr(got), bias_mode=bias_mode)


def test_resident_forward_non_finite_inputs():
    """Infinities and NaN reach exactly the outputs whose lists hold their neuron: the list padding reads a row
    of zeros, not another input."""
    import torch

    import paper_1708_02937_amd as sd

    p = _problem(1500, 70, 1, [3, 9, 30], 5)
    p.y0_dense[::3, ::17] = math.inf
    p.y0_dense[1::3, ::23] = math.nan
    p.y0_dense[:, 0] = math.inf
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    got = net.forward_dense(y).cpu().numpy()
    net.set_profiling(True)
    want = net.forward_dense(y).cpu().numpy()
    net.free()
    assert np.array_equal(got, want, equal_nan=True) and np.isfinite(got).any() and not np.isfinite(got).all()


def test_resident_forward_named_in_profiling_log():
    """A layer of 2^24 products or more is timed as a launch of its own under the resident kernel's name."""
    import torch

    import paper_1708_02937_amd as sd

    p = make_config(2, 0.01, L=2, batch=128)
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    want = net.forward_dense(y)
    net.set_profiling(True)
    got = net.forward_dense(y)
    rec = net.read_profile()
    net.free()
    assert [(k, name) for k, name, _ in rec] == [(0, "spmm_resident_kernel"), (1, "spmm_resident_kernel")]
    assert torch.equal(got, want)


@pytest.mark.parametrize("n,batch,L,lengths,bias_mode", [c for c in CASES if c[2] > 1] + [
    (40, 4096, 2, [3, 9], 0), (40, 4097, 2, [3, 9], 1), (33, 16384, 2, [5], 0), (33, 16385, 2, [5], 0)])
def test_resident_csr_forward(n, batch, L, lengths, bias_mode):
    """A dense enough CSR batch is placed into LDS by the product itself, and the result's row counts come from its
    last launch (row pointers in one workgroup up to 16384 rows, by the general scan beyond); empty rows among them."""
    import paper_1708_02937_amd as sd

    p = _problem(n, batch, L, lengths, n + batch)
    p.y0_dense[::7] = 0.0
    print("[case] resident csr", n, batch, L, bias_mode, flush=True)
    net = sd.net_from_problem(p, bias_mode=bias_mode)
    got = tuple(x.cpu().numpy() for x in net.forward_csr(*p.y0_as_csr()))
    net.free()
    parity.compare(p, got, bias_mode=bias_mode)


@pytest.mark.parametrize("batch", [3, 300, 1030])
def test_resident_csr_forward_checks_its_input(batch):
    """Row extents and columns out of range are reported, whichever sample of a workgroup's they are in, and rows
    that are all empty need no column or value array."""
    import paper_1708_02937_amd as sd

    p = _problem(500, batch, 2, [3, 9], 4)
    net = sd.net_from_problem(p)
    rp, c, v = p.y0_as_csr()
    for r in (0, 1, batch // 2, batch - 1):
        for at, wrong in ((rp[r], -1), (rp[r + 1] - 1, p.n), (rp[r], 1 << 30)):
            bad = c.copy()
            bad[at] = wrong
            print("[case] resident csr check", batch, r, wrong, flush=True)
            with pytest.raises(sd.SdnnError) as e:
                net.forward_csr(rp, bad, v)
            assert e.value.name == "SDNN_ERR_INVALID_INDEX"
    bad = rp.copy()
    bad[1] = bad[2] + 1
    with pytest.raises(sd.SdnnError) as e:
        net.forward_csr(bad, c, v)
    assert e.value.name == "SDNN_ERR_INVALID_INDEX"
    got = tuple(x.cpu().numpy() for x in net.forward_csr(rp, c, v))
    parity.compare(p, got)
    p.y0_dense[:] = 0.0
    got = tuple(x.cpu().numpy() for x in net.forward_csr(np.zeros(batch + 1, np.int64), c[:0], v[:0]))
    net.free()
    parity.compare(p, got)


@pytest.mark.parametrize("n,batch,d", [(1000, 125, 0.6), (1000, 129, 0.6), (3000, 253, 0.3), (4100, 131, 0.5),
                                       (2049, 1, 0.99), (600, 1027, 0.9)])
def test_high_fan_in_ragged_batches(n, batch, d):
    """Layers of density 2/9 and more at batches that are no multiple of four: the resident product or, with the batch
    rounded up inside the workspace, the LDS-tiled one; one row per sample compared, integer values bit for bit."""
    import torch

    import paper_1708_02937_amd as sd
    from workloads import integer_shadow, tiny_random

    p = tiny_random(n, n, 1, batch, w_density=d, y_density=0.7, dense_input=True, bias_lo=-1.0, bias_hi=1.0)
    p = integer_shadow(p)
    net = sd.net_from_problem(p)
    print("[case] high fan-in ragged", n, batch, d, flush=True)
    y = torch.from_numpy(p.y0_dense).cuda()
    got = net.forward_dense(y).cpu().numpy()
    net.set_profiling(True)
    other = net.forward_dense(y).cpu().numpy()
    net.free()
    assert got.tobytes() == other.tobytes()
    rows = np.arange(0, batch, 1 + batch // 40)
    parity.compare(p, dense_to_csr(got[rows]), rows=rows, exact=True)


@pytest.mark.parametrize("n,batch", [(5120, 1), (6000, 5), (9001, 33), (8200, 259), (12000, 331)])
def test_wide_layers_ragged_batches(n, batch):
    """Layers too wide for the resident product at batches that are no multiple of four (rounded up inside the
    workspace), dense and CSR input, and on the fixed scratch array."""
    import torch

    import paper_1708_02937_amd as sd

    p = _problem(n, batch, 2, [60, 0, 90, 64], n)
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    print("[case] wide ragged", n, batch, flush=True)
    got = net.forward_dense(y)
    parity.compare(p, dense_to_csr(got.cpu().numpy()))
    parity.compare(p, tuple(x.cpu().numpy() for x in net.forward_csr(*p.y0_as_csr())))
    out = torch.empty_like(y)
    sd.sdnn_forward_dense_noalloc(net.handle, 0, p.L, batch, y, out, sd.SDNN_ARM_SPARSE)
    assert torch.equal(out, got)
    net.free()


def test_scratch_array_without_room_for_rounding():
    """The fixed scratch array takes a batch whose two buffers fit only without the batch rounded up to four: the
    products then run at the batch as it is."""
    import torch

    import paper_1708_02937_amd as sd

    n = 40009
    batch = sd.sdnn_noalloc_scratch_bytes() // (2 * 4 * n)
    assert batch % 4 == 1 and 2 * 4 * n * (batch + 3) > sd.sdnn_noalloc_scratch_bytes()
    p = _problem(n, batch, 1, [3, 0, 5], 8)
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    print("[case] scratch array", n, batch, flush=True)
    out = torch.empty_like(y)
    sd.sdnn_forward_dense_noalloc(net.handle, 0, 1, batch, y, out, sd.SDNN_ARM_SPARSE)
    assert torch.equal(out, net.forward_dense(y))
    net.free()


@pytest.mark.parametrize("n,batch,lists,want", [
    (5200, 125, 0.25, "spmm_fanin_kernel"), (5200, 391, 0.25, "spmm_slots_kernel"), (5200, 251, 0.5, "spmm_slots_kernel"),
    (6000, 7, [20], "spmm_narrow_kernel"), (6000, 7, [20] * 5999 + [3000], "spmm_fanin_kernel"),
    (9000, 131, [10] * 4499 + [4000], "spmm_fanin_kernel"), (24000, 97, [32], "spmm_fanin_kernel"),
    (24000, 61, [32], "spmm_narrow_kernel")])
def test_ragged_batches_rounded_where_it_is_cheaper(n, batch, lists, want):
    """A batch that is no multiple of four is rounded up for the LDS-tiled product or the narrow-chunk gather only where
    they are the cheaper ones, and stays as it is on the plain gather otherwise: few samples at densities of a quarter, one
    list of thousands of entries, a mostly empty last chunk of 64 samples on wide layers."""
    import torch

    import paper_1708_02937_amd as sd
    from workloads import tiny_random

    if isinstance(lists, float):
        p = tiny_random(n, n, 1, batch, w_density=lists, y_density=0.7, dense_input=True)
    else:
        p = _problem(n, batch, 1, lists, n)
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    print("[case] ragged route", n, batch, want, flush=True)
    net.set_profiling(True)
    got = net.forward_dense(y).cpu().numpy()
    assert [name for _, name, _ in net.read_profile()][1:-1] == [want]
    out = torch.empty_like(y)
    sd.sdnn_forward_dense_noalloc(net.handle, 0, 1, batch, y, out, sd.SDNN_ARM_SPARSE)
    assert out.cpu().numpy().tobytes() == got.tobytes()
    net.free()
    rows = np.arange(0, batch, 1 + batch // 16)
    parity.compare(p, dense_to_csr(got[rows]), rows=rows)


@pytest.mark.parametrize("lists,want", [([10] * 699 + [700], "spmm_fanin_kernel"), ([20], "spmm_resident_kernel")])
def test_one_long_list_is_priced(lists, want):
    """One list of all 700 inputs among lists of 10: the wave that walks it sets the resident product's time in every
    round of workgroups, and the gather's once; without it the resident product is the cheaper one."""
    import torch

    import paper_1708_02937_amd as sd

    batch = 3000
    p = _problem(700, batch, 1, lists, 1)
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    print("[case] one long list", want, flush=True)
    got = net.forward_dense(y).cpu().numpy()
    net.set_profiling(True)
    logged = net.forward_dense(y).cpu().numpy()
    assert want in [name for _, name, _ in net.read_profile()]
    net.free()
    assert got.tobytes() == logged.tobytes()
    rows = np.arange(0, batch, 37)
    parity.compare(p, dense_to_csr(got[rows]), rows=rows)


@pytest.mark.parametrize("n,batch,L,lengths", [(157, 3667, 5, [1] * 156 + [78]), (2918, 301, 2, [10] * 700 + [1459]),
                                               (5000, 13, 2, [10] * 249 + [1000]), (4339, 85, 2, [10] * 130 + [2170])])
def test_few_long_lists(n, batch, L, lengths):
    """A few lists far longer than the rest, on whichever products they are priced into: dense and CSR input against the
    oracle, max.+ against numpy."""
    import torch

    import paper_1708_02937_amd as sd
    from workloads import csr_rows

    p = _problem(n, batch, L, lengths, n)
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    print("[case] few long lists", n, batch, L, flush=True)
    rows = np.arange(0, batch, 1 + batch // 64)
    parity.compare(p, dense_to_csr(net.forward_dense(y).cpu().numpy()[rows]), rows=rows)
    csr = tuple(x.cpu().numpy() for x in net.forward_csr(*p.y0_as_csr()))
    parity.compare(p, csr_rows(csr, rows), rows=rows)
    z = net.mxm(0, sd.SDNN_SEMIRING_MAX_PLUS, y).cpu().numpy()
    net.free()
    l = p.layers[0]
    i = np.repeat(np.arange(n), np.diff(l.row_ptr))
    for r in (0, batch // 2, batch - 1):
        want = np.full(n, -np.inf, dtype=np.float32)
        np.maximum.at(want, l.col, p.y0_dense[r, i] + l.val)
        assert np.array_equal(z[r], want)
