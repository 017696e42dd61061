"""GPU parity of the SpMV that has x come by in parts through LDS: where its parts, its
rounds and its workgroups' rows have edges (x of exactly so many parts and one entry more,
one to four tiles per wavefront, tile height 16, rows across several workgroups, empty
rows, the incomplete tile, x at an odd address), and that columns it is not for are left
to the general kernel.  Every test asks the library which kernel it is about."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_05032_amd import binding as B
from paper_1503_05032_amd import workloads as wl

from gpu_util import DeviceCsr, check_format, check_spmv, convert, second_kernel_ms

pytestmark = pytest.mark.gpu

PART = 79 * 1024 // 8          # entries of x in a part


def _rows(m, length, n, seed, mixed):
    """m rows of `length` random columns; mixed: a tenth of them empty, a third short, and
    one in the middle and one at the end that cross many tiles."""
    lens = np.full(m, length)
    if mixed:
        rng = np.random.default_rng(seed)
        u = rng.random(m)
        lens[u < 0.1] = 0
        lens[(u >= 0.1) & (u < 0.4)] = rng.integers(1, 9, size=int(((u >= 0.1) & (u < 0.4)).sum()))
        lens[m // 2] = min(n - 1, 30_000)
        lens[-1] = min(n - 1, 20_000)
    return wl.from_row_lengths(lens, n, seed=seed, name=f"rows{m}x{length}")


@pytest.mark.parametrize("m,length,n,sigma,mixed,tiles", [
    (17_000, 100, 30_000, 0, False, 1),            # 3320 tiles: one per wavefront
    (36_000, 101, 30_001, 0, True, 2),             # short and long rows
    (20_011, 150, 2 * PART, 0, False, 2), (20_011, 150, 2 * PART + 1, 0, False, 2),    # two parts and a little more
    (30_011, 201, 60_013, 0, False, 3), (50_000, 201, 60_013, 0, True, 3),
    (41_000, 201, 4 * PART, 0, False, 2), (66_000, 201, 4 * PART - 1, 0, True, 2),     # two rounds
    (20_000, 201, 5 * PART, 16, False, 1), (50_000, 201, 45_000, 16, True, 2), (40_000, 201, 20_000, 16, False, 1)])      # height 16; the last in two rounds
def test_parity(m, length, n, sigma, mixed, tiles):
    a = _rows(m, length, n, seed=m % 97, mixed=mixed)
    print("staged", m, length, n, sigma, mixed, a.nnz, flush=True)
    d = DeviceCsr(a)
    h = convert(d, sigma=sigma)
    check_format(d, h, a.name)
    assert B.csr5_get_form(h) == {"kernel": B.CSR5_KERNEL_PARTS, "wave_tiles": tiles, "plain": 0}
    info, first = B.csr5_get_info(h), None
    whole_tiles = info["p_complete"] * 64 * info["sigma"]
    fixed = int(np.searchsorted(a.row_ptr, whole_tiles, side="right")) - 1      # rows in the incomplete tile are added in any order
    for call in range(10):                         # the meeting words come back to rest
        check_spmv(d, h, (a.name, call))
        first = d.y.clone() if first is None else first
        assert torch.equal(d.y[:fixed], first[:fixed]), (a.name, call)
    assert second_kernel_ms(h, d.x, d.y) < 1e-3, a.name
    whole = torch.empty(n + 1, dtype=torch.float64, device="cuda:0")            # x at an odd address
    whole[1:] = d.x
    B.csr5_spmv_ex(h, whole[1:], d.y)
    torch.cuda.synchronize()
    assert torch.equal(d.y[:fixed], first[:fixed]), a.name
    d.y.fill_(float("nan"))                        # the entry point with its own cross-tile array: the general kernel
    B.csr5_spmv_static(h, d.x, d.y)
    torch.cuda.synchronize()
    _, s = oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, a.x)
    assert np.all(np.abs((d.y - first).cpu().numpy()[:a.m]) <= 2e-12 * s + 1e-300)
    B.csr5_free(h)


@pytest.mark.parametrize("m,length,n,sigma,tiles", [
    (28_000, 100, 2 * 2 * PART + 3, 0, 1), (30_011, 201, 60_013, 0, 2), (62_000, 145, 60_000, 0, 3), (92_000, 145, 60_000, 0, 4),
    (110_000, 145, 60_000, 0, 3),                  # two rounds
    (30_011, 201, 60_013, 16, 1), (50_000, 201, 60_001, 16, 2)])
def test_single_precision(m, length, n, sigma, tiles):
    a = _rows(m, length, n, seed=5, mixed=True)
    d = DeviceCsr(a)
    val, x = d.val.float(), d.x.float()
    products = val.double() * x.double()[d.col_idx.long()]
    want = torch.segment_reduce(products, "sum", offsets=d.row_ptr.long(), initial=0)
    scale = torch.segment_reduce(products.abs(), "sum", offsets=d.row_ptr.long(), initial=0)
    y = torch.empty(a.m, dtype=torch.float32, device="cuda:0")
    h = B.csr5s_convert_ex(a.m, a.n, a.nnz, d.row_ptr, d.col_idx, val, sigma=sigma)
    assert B.csr5_get_form(h) == {"kernel": B.CSR5_KERNEL_PARTS, "wave_tiles": tiles, "plain": 0}
    for call in range(10):
        y.fill_(float("nan"))
        B.csr5s_spmv_ex(h, x, y)
        assert bool(((y.double() - want).abs() <= 1e-5 * scale + 1e-30).all()), call      # at most 64 additions per term: 64 * 2^-24 = 3.8e-6
    B.csr5_free(h)


def test_nan_and_infinities_of_x_reach_their_rows_only():
    a = _rows(30_011, 201, 60_013, seed=3, mixed=False)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_PARTS
    x = a.x.copy()
    x[[0, PART - 1, PART, 60_012]] = [np.nan, np.inf, -np.inf, np.nan]
    d.x = torch.from_numpy(x).cuda()
    B.csr5_spmv_ex(h, d.x, d.y)
    torch.cuda.synchronize()
    y, (want, s) = d.y.cpu().numpy(), oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, x)
    odd = ~np.isfinite(want)
    assert 0 < odd.sum() < a.m and np.array_equal(np.isnan(y), np.isnan(want)) and np.array_equal(y[odd & ~np.isnan(want)], want[odd & ~np.isnan(want)])
    assert np.all(np.abs(y[~odd] - want[~odd]) <= 1e-12 * s[~odd] + 1e-300)
    B.csr5_free(h)


def _columns(kind, m, length, n, rng):
    if kind == "band":                             # random, but near the row's own place
        return (np.arange(m)[:, None] * n // m + rng.integers(-1000, 1000, size=(m, length))).clip(0, n - 1)
    if kind == "popular":                          # a few columns hold most entries
        return rng.permutation(n)[np.minimum((rng.pareto(0.7, size=(m, length))).astype(np.int64), n - 1)]
    return rng.integers(0, n - length, size=m)[:, None] + np.arange(length)[None]      # runs


@pytest.mark.parametrize("kind", ["band", "popular", "runs"])
def test_other_columns_take_the_general_kernel(kind):
    m, length, n = 25_000, 201, 40_000
    a = wl.from_row_lengths(np.full(m, length), n, seed=2, name=kind)
    a.col_idx[:] = np.sort(_columns(kind, m, length, n, np.random.default_rng(4)), axis=1).reshape(-1)      # (columns may repeat)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_TILES
    check_spmv(d, h, kind)
    assert second_kernel_ms(h, d.x, d.y) > 1e-3, kind
    B.csr5_free(h)


def test_graph_replays():
    a = _rows(30_011, 201, 60_013, seed=9, mixed=True)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_PARTS
    check_spmv(d, h, "eager")
    want = d.y.clone()[:-2000]                     # (not the rows in the incomplete tile, which are added in any order)
    yg = torch.empty_like(d.y)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.csr5_spmv_ex(h, d.x, yg)
    for replay in range(4):
        yg.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(yg[:-2000], want), replay
        B.csr5_spmv_ex(h, d.x, d.y)
        torch.cuda.synchronize()
        assert torch.equal(d.y[:-2000], want), replay
    B.csr5_free(h)
