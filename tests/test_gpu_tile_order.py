"""GPU parity of the tile order by columns: matrices most of whose tiles lie inside one
long row, with x larger than the L2 of one accelerator die, at the sizes where the order
begins (2048 complete tiles; x of 4 MiB) and at workgroups of four and of two tiles."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_05032_amd import binding as B
from paper_1503_05032_amd import workloads as wl

from gpu_util import DeviceCsr, check_format, check_spmv, convert, second_kernel_ms

pytestmark = pytest.mark.gpu


def _matrix(sigma, tiles, ragged, n, seed):
    """`tiles` complete tiles and `ragged` further entries: rows of 5 to 20 tiles, a fifth
    of the entries in short and empty rows between them."""
    rng = np.random.default_rng(seed)
    T = 64 * sigma
    total, lens = tiles * T + ragged, []
    while total > 0:
        for k in [int(rng.integers(5 * T, 20 * T))] + rng.integers(0, 9, size=600).tolist():
            k = min(k, total)
            lens.append(k)
            total -= k
    return wl.from_row_lengths(np.array(lens), n, seed=seed, name=f"long{sigma}_{tiles}")


@pytest.mark.parametrize("sigma,tiles,ragged,wide", [(8, 2048, 0, False), (8, 2047, 511, False), (8, 2049, 1, True), (8, 3001, 77, False),
                                                     (16, 2050, 3, False), (17, 2051, 500, True), (32, 2048, 9, False)])
def test_long_rows_with_a_large_x(sigma, tiles, ragged, wide):
    for n in (524_287, 524_288, 700_001):
        a = _matrix(sigma, tiles, ragged, n, seed=sigma + tiles)
        print("order", sigma, tiles, ragged, wide, n, a.m, a.nnz, flush=True)
        d = DeviceCsr(a, wide=wide)
        h = convert(d, sigma=sigma)
        if n == 700_001:
            check_format(d, h, (a.name, n))
        for call in range(2):
            check_spmv(d, h, (a.name, n, call), x=np.random.default_rng(call).standard_normal(n))
        # by column means two kernels; by number matrices of this size and form are one
        assert (second_kernel_ms(h, d.x, d.y) > 1e-3) == (tiles >= 2048 and n >= 524_288), (a.name, n)
        if not wide:                                     # the entry point with its own cross-tile array takes the same order
            y = d.y.clone()
            d.y.fill_(float("nan"))
            B.csr5_spmv_static(h, d.x, d.y)
            torch.cuda.synchronize()
            _, s = oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, d.x.cpu().numpy())
            assert np.all(np.abs((y - d.y).cpu().numpy()) <= 2e-12 * s + 1e-300)
        B.csr5_to_csr(h)
        torch.cuda.synchronize()
        assert np.array_equal(d.col_idx.cpu().numpy(), a.col_idx)
        B.csr5_free(h)


def test_long_rows_single_precision():
    a = _matrix(16, 2100, 5, 1_100_000, seed=3)
    d = DeviceCsr(a)
    val, x = d.val.float(), d.x.float()
    y = torch.full((a.m,), float("nan"), dtype=torch.float32, device="cuda:0")
    h = B.csr5s_convert_ex(a.m, a.n, a.nnz, d.row_ptr, d.col_idx, val, sigma=16)
    B.csr5s_spmv_ex(h, x, y)
    torch.cuda.synchronize()
    assert min(B.csr5s_spmv_profile(h, x, y, reps=100)[1] for _ in range(2)) > 1e-3      # by column: two kernels
    torch.cuda.synchronize()
    ref, s = oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val.astype(np.float32).astype(np.float64), x.cpu().numpy().astype(np.float64))
    # a term passes through the walk, the tile's scan and the sum over a row's 20 tiles at most: fewer than 64 additions of 2^-24 each
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 1e-5 * s + 1e-30)
    B.csr5_free(h)


@pytest.mark.parametrize("sigma,tiles,long", [(8, 2050, 0), (16, 6200, 0), (8, 8_000, 690_000), (16, 5_500, 690_000)])
def test_long_rows_same_bits_on_every_call(sigma, tiles, long):
    """A matrix taken by column that would otherwise be one kernel (short rows on average, or at most 6144 tiles)
    returns the same bits on every call: rows of 5 to 20 tiles, cut by the 64-tile stretches of the second kernel,
    and one of `long` entries (1347 and 673 tiles: its sum takes 16 * 64 tiles at a time).  No incomplete tile: its
    rows are summed atomically."""
    a = _matrix(sigma, tiles, 0, 700_001, seed=tiles)
    if long:                                             # some hundred rows in the middle become one
        lens = np.diff(a.row_ptr).astype(np.int64)
        at = len(lens) // 2
        end = at + int(np.searchsorted(np.cumsum(lens[at:]), long))
        lens = np.concatenate([lens[:at], [lens[at:end].sum()], lens[end:]])
        assert lens.max() > 2 * 64 * 64 * sigma
        a = wl.from_row_lengths(lens, 700_001, seed=1, name="one_long")
    assert a.nnz == tiles * 64 * sigma
    d = DeviceCsr(a)
    h = convert(d, sigma=sigma)
    check_spmv(d, h, (a.name, tiles))
    first = d.y.clone()
    for call in range(30):
        for spmv in (B.csr5_spmv_ex, B.csr5_spmv_static):
            d.y.fill_(float("nan"))
            spmv(h, d.x, d.y)
            assert torch.equal(d.y, first), (call, int((d.y != first).sum()))
    B.csr5_free(h)


def _low_columns(sigma, tiles, share, n):
    """As _matrix, but in a first `share` of the matrix all columns lie in the lowest sixteenth of n."""
    a = _matrix(sigma, tiles, 0, n // 16, seed=int(100 * share))
    rows = np.repeat(np.arange(a.m), np.diff(a.row_ptr))
    spread = np.arange(a.nnz) >= share * a.nnz
    spread = spread[a.row_ptr[rows]]                     # whole rows
    col = np.where(spread, a.col_idx.astype(np.int64) * 16, a.col_idx).astype(np.int32)
    x = np.random.default_rng(1).standard_normal(n)
    return wl.Csr(a.m, n, a.row_ptr, col, a.val, x, f"low{share}")


@pytest.mark.parametrize("sigma,tiles", [(8, 2060), (8, 6000), (16, 2500)])
@pytest.mark.parametrize("share", [0.0, 0.3, 0.55, 0.85, 1.0])
def test_crowded_columns_are_taken_by_number(sigma, tiles, share):
    """More than three quarters of the tiles inside one row beginning in an eighth of the columns (the fullest 128 of
    1024 buckets): by number, as one kernel.  The low sixteenth is 64 buckets; the 64 fullest of the other 960 hold
    at most 4 of the (1 - share) * 2060 tiles spread over them each, 0.12 of all: 0.55 stays below 0.75."""
    a = _low_columns(sigma, tiles, share, 700_000)
    d = DeviceCsr(a)
    h = convert(d, sigma=sigma)
    check_spmv(d, h, (a.name, sigma, tiles))
    assert (second_kernel_ms(h, d.x, d.y) > 1e-3) == (share < 0.75)
    B.csr5_free(h)


def test_sort_of_many_tiles():
    """127 k tiles (the scan over several workgroups, 124 slices of the sort): results, and the sort beside the
    conversion, of which one workgroup for all tiles made 200 us."""
    L, m, n, sigma = 20_000, 3250, 600_000, 8
    g = torch.Generator(device="cuda:0")
    g.manual_seed(7)
    u = torch.rand((m, L), generator=g, device="cuda:0", dtype=torch.float64)
    col = ((torch.arange(L, device="cuda:0") + u) * (n / L)).long().clamp_(max=n - 1).to(torch.int32).flatten()
    val = torch.rand(m * L, generator=g, device="cuda:0", dtype=torch.float64) - 0.5
    x = torch.rand(n, generator=g, device="cuda:0", dtype=torch.float64) - 0.5
    row_ptr = torch.arange(m + 1, device="cuda:0", dtype=torch.int32) * L
    products = (val * x[col.long()]).view(m, L)
    ref, s = products.sum(1), products.abs().sum(1)
    before = col.clone()
    ws = torch.empty(B.csr5_workspace_bytes(m, m * L, sigma), dtype=torch.uint8, device="cuda:0")
    y = torch.empty(m, dtype=torch.float64, device="cuda:0")
    ms = {0: [], B.CSR5_FLAG_NO_HOST_CHECK: []}
    for call in range(6):
        for flags in ms:
            t0, t1 = torch.cuda.Event(True), torch.cuda.Event(True)
            t0.record()
            h = B.csr5_convert_ex(m, n, m * L, row_ptr, col, val, sigma=sigma, workspace=ws, flags=flags)
            t1.record()
            y.fill_(float("nan"))
            B.csr5_spmv_ex(h, x, y)
            torch.cuda.synchronize()
            ms[flags].append(t0.elapsed_time(t1))
            assert bool(((y - ref).abs() <= 1e-12 * s).all())
            B.csr5_to_csr(h)
            torch.cuda.synchronize()
            B.csr5_free(h)
            assert torch.equal(col, before)
    print("blocking, enqueued (ms):", *(min(v) for v in ms.values()))
    assert min(ms[0]) < min(ms[B.CSR5_FLAG_NO_HOST_CHECK]) + 0.1


def test_only_a_blocking_conversion_lays_out_the_order():
    """After CSR5_FLAG_NO_HOST_CHECK the matrix keeps its other form, also once csr5_status has been called."""
    a = _matrix(8, 2100, 5, 700_001, seed=11)
    for flags, two in ((B.CSR5_FLAG_NONE, True), (B.CSR5_FLAG_NO_HOST_CHECK, False), (B.CSR5_FLAG_AUX_ONE_KERNEL, False),
                       (B.CSR5_FLAG_AUX_TWO_KERNELS, True)):
        d = DeviceCsr(a)
        h = convert(d, sigma=8, flags=flags)
        check_spmv(d, h, (a.name, flags))
        assert B.csr5_status(h) & 3 == 0
        check_spmv(d, h, (a.name, flags))
        assert (second_kernel_ms(h, d.x, d.y) > 1e-3) == two, flags
        B.csr5_free(h)
