"""GPU parity of the SpMV that keeps the part of x around the diagonal in LDS: x just above
the window and a little more, tall and wide matrices, entries in and outside the window,
rows across several workgroups and empty ones, both tile heights, one and two kernels, x
at an odd address; and which columns are left to the general kernel.  Every test asks the
library which kernel it is about."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_05032_amd import binding as B
from paper_1503_05032_amd import workloads as wl

from gpu_util import DeviceCsr, check_format, check_spmv, convert, second_kernel_ms

pytestmark = pytest.mark.gpu

WINDOW = 78 * 1024 // 8        # entries of x in a window


def _band(m, n, lo, hi, w, far=0.0, uneven=False, seed=0):
    """Rows of lo to hi entries within +-w columns of the diagonal, a share `far` of them
    anywhere; uneven: a tenth of the rows empty, one in the middle and the last one long."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(lo, hi + 1, size=m)
    if uneven:
        lens[rng.random(m) < 0.1] = 0
        lens[m // 2], lens[-1] = 30_000, 20_000
    row_ptr = np.zeros(m + 1, dtype=np.int32)
    np.cumsum(lens, out=row_ptr[1:])
    rows = np.repeat(np.arange(m, dtype=np.int64), lens)
    col = (rows * n // m + rng.integers(-w, w + 1, size=rows.size)).clip(0, n - 1)
    if far:
        col = np.where(rng.random(rows.size) < far, rng.integers(0, n, size=rows.size), col)
    col = (np.sort(rows * n + col) - rows * n).astype(np.int32)                 # (columns may repeat)
    return wl.Csr(m=m, n=n, row_ptr=row_ptr, col_idx=col, val=rng.uniform(-1, 1, rows.size), x=rng.uniform(-1, 1, n), name=f"band{m}x{w}")


@pytest.mark.parametrize("m,n,lo,hi,w,far,sigma,uneven", [
    (20_000, WINDOW + 1, 165, 215, 4000, 0.0, 0, False),           # x of one window and an entry
    (20_000, WINDOW + 17, 165, 215, 4000, 0.0, 0, True),
    (20_001, 90_003, 165, 215, 5000, 0.0, 0, False),               # wide
    (430_003, 100_001, 5, 13, 5000, 0.1, 0, True),                # tall
    (20_000, 300_000, 165, 215, 7000, 0.1, 0, True),              # a band wider than the window
    (20_000, 200_000, 200, 200, 5000, 0.4, 0, False),             # rows of one length, many entries elsewhere
    (45_000, 90_000, 165, 215, 5000, 0.2, 16, True),               # height 16
    (110_000, 200_001, 165, 215, 5000, 0.1, 8, True)])            # more than 32768 tiles: two kernels
def test_parity(m, n, lo, hi, w, far, sigma, uneven):
    a = _band(m, n, lo, hi, w, far, uneven, seed=m % 97)
    print("window", m, n, lo, hi, w, far, sigma, uneven, a.nnz, flush=True)
    d = DeviceCsr(a)
    h = convert(d, sigma=sigma)
    check_format(d, h, a.name)
    info, first = B.csr5_get_info(h), None
    assert B.csr5_get_form(h) == {"kernel": B.CSR5_KERNEL_WINDOW, "wave_tiles": 2 if info["sigma"] == 8 else 1, "plain": 0}
    one = info["p"] <= 32768
    assert one == (m < 100_000 or lo < 160), info["p"]
    whole_tiles = info["p_complete"] * 64 * info["sigma"]
    fixed = int(np.searchsorted(a.row_ptr, whole_tiles, side="right")) - 1      # rows in the incomplete tile are added in any order
    for call in range(10):                         # the meeting words come back to rest
        check_spmv(d, h, (a.name, call))
        first = d.y.clone() if first is None else first
        if one:
            assert torch.equal(d.y[:fixed], first[:fixed]), (a.name, call)
    assert (second_kernel_ms(h, d.x, d.y) < 1e-3) == one, a.name
    _, s = oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, a.x)
    whole = torch.empty(n + 1, dtype=torch.float64, device="cuda:0")            # x at an odd address
    whole[1:] = d.x
    d.y.fill_(float("nan"))
    B.csr5_spmv_ex(h, whole[1:], d.y)
    torch.cuda.synchronize()
    assert np.all(np.abs((d.y - first).cpu().numpy()) <= 2e-12 * s + 1e-300)
    d.y.fill_(float("nan"))                        # the entry point with its own cross-tile array: two kernels
    B.csr5_spmv_static(h, d.x, d.y)
    torch.cuda.synchronize()
    assert np.all(np.abs((d.y - first).cpu().numpy()) <= 2e-12 * s + 1e-300)
    B.csr5_free(h)


def _single(a, sigma, kernel, calls=10):
    """Products in single precision against sums in double precision; the form is the one named."""
    d = DeviceCsr(a)
    val, x = d.val.float(), d.x.float()
    products = val.double() * x.double()[d.col_idx.long()]
    want = torch.segment_reduce(products, "sum", offsets=d.row_ptr.long(), initial=0)
    scale = torch.segment_reduce(products.abs(), "sum", offsets=d.row_ptr.long(), initial=0)
    y = torch.empty(a.m, dtype=torch.float32, device="cuda:0")
    h = B.csr5s_convert_ex(a.m, a.n, a.nnz, d.row_ptr, d.col_idx, val, sigma=sigma)
    assert B.csr5_get_form(h)["kernel"] == kernel, B.csr5_get_form(h)
    for call in range(calls):
        y.fill_(float("nan"))
        B.csr5s_spmv_ex(h, x, y)
        assert bool(((y.double() - want).abs() <= 1e-5 * scale + 1e-30).all()), call      # at most 64 additions per term: 64 * 2^-24 = 3.8e-6
    B.csr5_free(h)


@pytest.mark.parametrize("m,n,sigma,w,far", [
    (60_000, 2 * WINDOW + 1, 0, 4000, 0.0),                        # x of one window and an entry
    (60_000, 150_001, 0, 5000, 0.0), (70_000, 150_001, 0, 5000, 0.1),
    (110_000, 150_001, 16, 9500, 0.1),                             # height 16; a band as wide as the window
    (300_000, 400_003, 8, 9500, 0.05)])                            # more than 32768 tiles: two kernels
def test_single_precision(m, n, sigma, w, far):
    _single(_band(m, n, 60, 110, w, far, True, seed=5), sigma, B.CSR5_KERNEL_WINDOW)


@pytest.mark.parametrize("m,lo,hi,w,far,single,kernel", [
    (50_000, 165, 215, 5000, 0.2, False, B.CSR5_KERNEL_WINDOW),       # two rounds of 6 parts, 2 M entries elsewhere
    (50_000, 60, 110, 5000, 0.2, False, B.CSR5_KERNEL_PARTS),         # one round
    (100_000, 60, 110, 7000, 0.1, True, B.CSR5_KERNEL_WINDOW),
    (70_000, 60, 110, 7000, 0.3, True, B.CSR5_KERNEL_PARTS)])
def test_bands_that_either_form_may_have(m, lo, hi, w, far, single, kernel):
    a = _band(m, m, lo, hi, w, far, seed=4)
    if single:
        return _single(a, 0, kernel)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == kernel, B.csr5_get_form(h)
    for call in range(3):
        check_spmv(d, h, call)
    B.csr5_free(h)


def test_nan_and_infinities_of_x_reach_their_rows_only():
    a = _band(40_001, 90_003, 60, 110, 5000, 0.1, seed=3)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_WINDOW
    x = a.x.copy()
    x[[0, WINDOW - 1, WINDOW, 90_002]] = [np.nan, np.inf, -np.inf, np.nan]
    d.x = torch.from_numpy(x).cuda()
    B.csr5_spmv_ex(h, d.x, d.y)
    torch.cuda.synchronize()
    y, (want, s) = d.y.cpu().numpy(), oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, x)
    odd = ~np.isfinite(want)
    assert 0 < odd.sum() < a.m and np.array_equal(np.isnan(y), np.isnan(want)) and np.array_equal(y[odd & ~np.isnan(want)], want[odd & ~np.isnan(want)])
    assert np.all(np.abs(y[~odd] - want[~odd]) <= 1e-12 * s[~odd] + 1e-300)
    B.csr5_free(h)


@pytest.mark.parametrize("w,far,n", [(500, 0.0, 400_000), (5000, 0.8, 2_000_000), (200_000, 0.0, 2_000_000)])
def test_other_columns_take_the_general_kernel(w, far, n):
    """A band that the L1 holds, one with too little in it, one far too wide."""
    a = _band(20_000, n, 200, 200, w, far, seed=2)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_TILES
    check_spmv(d, h, w)
    assert second_kernel_ms(h, d.x, d.y) > 1e-3, w
    B.csr5_free(h)


def test_graph_replays():
    a = _band(50_001, 90_003, 60, 110, 5000, 0.1, True, seed=9)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_WINDOW
    check_spmv(d, h, "eager")
    want = d.y.clone()[:-1]                        # (not the long row that ends in the incomplete tile)
    yg = torch.empty_like(d.y)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.csr5_spmv_ex(h, d.x, yg)
    for replay in range(4):
        yg.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(yg[:-1], want), replay
        B.csr5_spmv_ex(h, d.x, d.y)
        torch.cuda.synchronize()
        assert torch.equal(d.y[:-1], want), replay
    B.csr5_free(h)
