"""GPU parity of the SpMV that has the x of far entries gathered into a buffer by a kernel of its own: x at and
around the edges of the gathered blocks, with and without a window, tall and wide matrices, empty and long rows,
both tile heights, one and two kernels for the sums, several chunks; and which matrices are left alone.  Every
test asks the library which kernel it is about."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_05032_amd import binding as B
from paper_1503_05032_amd import workloads as wl

from gpu_util import DeviceCsr, check_format, check_spmv, convert, second_kernel_ms

pytestmark = pytest.mark.gpu

BLOCK = 128 * 1024 // 8        # entries of x in a block


def _far(m, n, lo, hi, near, uneven=False, seed=0, banded_from=1.0):
    """Rows of lo to hi entries, a share `near` of them within +-4000 columns of the diagonal, the others anywhere;
    uneven: a tenth of the rows empty, one in the middle and the last one long; banded_from: from that share of the rows on
    all are near."""
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    lens = torch.randint(lo, hi + 1, (m,), generator=g, device="cuda:0")
    if uneven:
        lens[torch.rand(m, generator=g, device="cuda:0") < 0.1] = 0
        lens[m // 2], lens[-1] = 30_000, 20_000
    rows = torch.repeat_interleave(torch.arange(m, device="cuda:0"), lens)
    col = torch.randint(0, n, rows.shape, generator=g, device="cuda:0")
    band = (rows * n // m + torch.randint(-4000, 4001, rows.shape, generator=g, device="cuda:0")).clamp_(0, n - 1)
    col = torch.where((torch.rand(rows.shape, generator=g, device="cuda:0") < near) | (rows >= banded_from * m), band, col)
    col[0], col[-1] = 0, n - 1
    col = (torch.sort(rows * n + col).values - rows * n).int()                  # (columns may repeat)
    row_ptr = torch.zeros(m + 1, dtype=torch.int64, device="cuda:0")
    torch.cumsum(lens, 0, out=row_ptr[1:])
    rng = np.random.default_rng(seed)
    return wl.Csr(m=m, n=n, row_ptr=row_ptr.int().cpu().numpy(), col_idx=col.cpu().numpy(), val=rng.uniform(-1, 1, rows.numel()),
                  x=rng.uniform(-1, 1, n), name=f"far{m}x{n}")


@pytest.mark.parametrize("m,n,lo,hi,near,sigma,uneven,one", [
    (820_000, 600 * BLOCK, 15, 25, 0.0, 8, False, True),       # whole blocks, no window, height 8
    (1_100_001, 200 * BLOCK + 1, 15, 25, 0.0, 0, True, True),
    (440_000, 300 * BLOCK - 1, 60, 100, 0.4, 16, True, True), # a window; height 16, one kernel for the sums
    (7_500_000, 200 * BLOCK + 17, 1, 6, 0.1, 0, True, True),  # tall
    (50_001, 8_000_001, 600, 800, 0.4, 16, True, True),        # wide, rows longer than half a tile, a window
    (1_300_000, 250 * BLOCK + 5, 30, 40, 0.45, 8, True, False),       # a window; more than 32768 tiles: a kernel more
    (1_300_000, 250 * BLOCK + 5, 18, 26, 0.15, 8, True, False),       # the same without
    (900_000, 1024 * BLOCK, 15, 25, 0.0, 0, False, True)])     # the largest x
def test_parity(m, n, lo, hi, near, sigma, uneven, one):
    a = _far(m, n, lo, hi, near, uneven, seed=m % 97)
    print("far", m, n, lo, hi, near, sigma, uneven, a.nnz, flush=True)
    d = DeviceCsr(a)
    h = convert(d, sigma=sigma, use_workspace=False)
    check_format(d, h, a.name)
    info, first = B.csr5_get_info(h), None
    assert B.csr5_get_form(h) == {"kernel": B.CSR5_KERNEL_GATHERED, "wave_tiles": 2 if info["sigma"] == 8 else 1, "plain": 0}
    assert one == (info["p"] <= 32768) and info["sigma"] == (sigma or 16), info
    whole_tiles = info["p_complete"] * 64 * info["sigma"]
    fixed = int(np.searchsorted(a.row_ptr, whole_tiles, side="right")) - 1      # rows in the incomplete tile are added in any order
    for call in range(6):                          # every one of the handle's buffers
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
    d.y.fill_(float("nan"))                        # the entry point that uses no buffer
    B.csr5_spmv_static(h, d.x, d.y)
    torch.cuda.synchronize()
    assert np.all(np.abs((d.y - first).cpu().numpy()) <= 2e-12 * s + 1e-300)
    B.csr5_to_csr(h)
    torch.cuda.synchronize()
    assert np.array_equal(d.col_idx.cpu().numpy(), a.col_idx) and np.array_equal(d.val.cpu().numpy(), a.val)
    B.csr5_free(h)


@pytest.mark.parametrize("m,n,lo,hi,near,sigma,single", [
    (1_100_000, 2 * 260 * BLOCK + 1, 15, 25, 0.0, 0, True), (1_100_000, 2 * 260 * BLOCK - 1, 30, 50, 0.45, 16, True),
    (3_000_000, 4_000_001, 25, 35, 0.45, 0, False),            # 45 M entries through the buffer, in two chunks
    (3_000_000, 4_000_001, 10, 20, 0.1, 0, False),             # 37 M entries through the buffer, in two chunks
    (3_000_000, 6_000_001, 20, 30, 0.05, 0, True)])             # 68 M, two chunks
def test_against_sums_in_double_precision(m, n, lo, hi, near, sigma, single):
    a = _far(m, n, lo, hi, near, True, seed=5)
    d = DeviceCsr(a)
    val, x = (d.val.float(), d.x.float()) if single else (d.val, d.x)
    products = val.double() * x.double()[d.col_idx.long()]
    want = torch.segment_reduce(products, "sum", offsets=d.row_ptr.long(), initial=0)
    scale = torch.segment_reduce(products.abs(), "sum", offsets=d.row_ptr.long(), initial=0)
    del products
    y = torch.empty(a.m, dtype=val.dtype, device="cuda:0")
    h = (B.csr5s_convert_ex if single else B.csr5_convert_ex)(a.m, a.n, a.nnz, d.row_ptr, d.col_idx, val, sigma=sigma)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED, B.csr5_get_form(h)
    # single precision: at most 64 additions per term, 64 * 2^-24 = 3.8e-6; double: the bar of gpu_util
    rel, tiny = (1e-5, 1e-30) if single else (1e-12, 1e-300)
    for call in range(5):
        y.fill_(float("nan"))
        (B.csr5s_spmv_ex if single else B.csr5_spmv_ex)(h, x, y)
        assert bool(((y.double() - want).abs() <= rel * scale + tiny).all()), call
    odd = torch.empty(a.n + 1, dtype=x.dtype, device="cuda:0")                  # x at an address that is no multiple of 16
    odd[1:] = x
    y.fill_(float("nan"))
    (B.csr5s_spmv_ex if single else B.csr5_spmv_ex)(h, odd[1:], y)
    assert bool(((y.double() - want).abs() <= rel * scale + tiny).all()), "odd"
    B.csr5_free(h)


def test_far_entries_in_a_part_of_the_rows():
    """64 M far entries among the first four fifths of the rows, in two chunks: the buffer is no larger than what it may be."""
    a = _far(5_000_000, 4_000_001, 15, 25, 0.2, seed=8, banded_from=0.8)
    d = DeviceCsr(a)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    h = B.csr5_convert_ex(a.m, a.n, a.nnz, d.row_ptr, d.col_idx, d.val)
    held = before - torch.cuda.mem_get_info()[0]
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED
    # workspace, lists and buffer, and not the 20 MB that the conversion counts in (the driver hands out 2 MB at a time)
    assert held <= B.csr5_workspace_bytes(a.m, a.nnz) + 8 * 0.64 * a.nnz * 1.01 + (256 << 20) + (8 << 20), held
    B.csr5_spmv_ex(h, d.x, d.y)
    first = d.y.clone()
    B.csr5_to_csr(h)
    products = d.val * d.x[d.col_idx.long()]
    want = torch.segment_reduce(products, "sum", offsets=d.row_ptr.long(), initial=0)
    scale = torch.segment_reduce(products.abs(), "sum", offsets=d.row_ptr.long(), initial=0)
    assert bool(((first - want).abs() <= 1e-12 * scale + 1e-300).all())
    B.csr5_free(h)


def test_left_alone_where_memory_is_short():
    """Lists and buffer of 350 MB, 1.2 GB free: more than an eighth of it.  Nothing beyond the workspace is held."""
    a = _far(1_100_000, 200 * BLOCK, 15, 25, 0.0, seed=2)
    d = DeviceCsr(a)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    fill = []
    for _ in range(2):                             # (what is free after a large allocation is more than was left)
        fill.append(torch.empty(max(torch.cuda.mem_get_info()[0] - (1200 << 20), 1 << 20), dtype=torch.uint8, device="cuda:0"))
    before = torch.cuda.mem_get_info()[0]
    assert before <= 1250 << 20, before
    for _ in range(3):
        h = convert(d, use_workspace=False)
        held = before - torch.cuda.mem_get_info()[0]
        assert B.csr5_get_form(h)["kernel"] != B.CSR5_KERNEL_GATHERED
        assert held <= B.csr5_workspace_bytes(a.m, a.nnz) + (8 << 20), held
        check_spmv(d, h, "short")
        B.csr5_to_csr(h)
        B.csr5_free(h)
    del fill
    torch.cuda.empty_cache()
    h = convert(d, use_workspace=False)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED
    check_spmv(d, h, "enough")
    B.csr5_free(h)


def test_release_with_a_product_in_flight():
    """csr5_free waits for the device before the buffer goes: the product that was enqueued is whole."""
    a = _far(1_100_001, 200 * BLOCK + 1, 15, 25, 0.1, seed=6)
    d = DeviceCsr(a)
    stream, col, val = torch.cuda.Stream(), d.col_idx.clone(), d.val.clone()
    for _ in range(3):
        d.col_idx.copy_(col)
        d.val.copy_(val)
        d.y.fill_(float("nan"))
        h = convert(d, use_workspace=False)
        assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED
        for _ in range(3):
            B.csr5_spmv_ex(h, d.x, d.y, stream=stream)
        B.csr5_free(h)
        y, (want, s) = d.y.cpu().numpy(), oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, a.x)
        assert np.all(np.abs(y - want) <= 1e-12 * s + 1e-300)


def test_products_in_flight_on_four_streams_and_other_vectors():
    a = _far(700_001, 200 * BLOCK + 1, 45, 55, 0.36, True, seed=3)
    d = DeviceCsr(a)
    h = convert(d, use_workspace=False)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED
    streams = [torch.cuda.Stream() for _ in range(4)]
    xs = [d.x, -d.x, d.x.flip(0).contiguous(), d.x * 3]
    want = []
    for x in xs:
        B.csr5_spmv_ex(h, x, d.y)
        want.append(d.y.clone())
    torch.cuda.synchronize()
    for call in range(3):
        ys = [torch.full_like(d.y, float("nan")) for _ in xs]
        torch.cuda.synchronize()
        for s, x, y in zip(streams, xs, ys):
            B.csr5_spmv_ex(h, x, y, stream=s)
        torch.cuda.synchronize()
        for y, w in zip(ys, want):
            assert torch.equal(y[:-1], w[:-1]), call        # (not the long row that ends in the incomplete tile)
    B.csr5_free(h)


def test_graph_replays():
    a = _far(900_001, 200 * BLOCK + 1, 25, 35, 0.2, True, seed=9)
    d = DeviceCsr(a)
    h = convert(d, use_workspace=False)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED
    check_spmv(d, h, "eager")
    want = d.y.clone()[:-1]                        # (not the long row that ends in the incomplete tile)
    _, s = oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, a.x)
    bar = torch.from_numpy(2e-12 * s + 1e-300).cuda()        # other kernels: either is within 1e-12 of the oracle
    yg = torch.empty_like(d.y)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert B.csr5_get_form(h)["kernel"] != B.CSR5_KERNEL_GATHERED
        B.csr5_spmv_ex(h, d.x, yg)
    for replay in range(4):
        yg.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert bool(((yg - d.y).abs() <= bar).all()), replay
        B.csr5_spmv_ex(h, d.x, d.y)
        torch.cuda.synchronize()
        assert torch.equal(d.y[:-1], want), replay
    B.csr5_free(h)


def test_more_products_in_flight_than_buffers_and_replays_beside_them():
    """Twelve products of one handle on six streams, each with an x of its own, and two graphs that are replayed beside
    them: no row is longer than a tile, so neither a product nor a replay needs anything of the handle to itself."""
    a = _far(1_100_001, 200 * BLOCK + 1, 15, 25, 0.1, seed=6)
    d = DeviceCsr(a)
    h = convert(d, use_workspace=False)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED
    info = B.csr5_get_info(h)
    fixed = int(np.searchsorted(a.row_ptr, info["p_complete"] * 64 * info["sigma"], side="right")) - 1      # rows in the incomplete tile are added in any order
    streams, side = [torch.cuda.Stream() for _ in range(6)], [torch.cuda.Stream() for _ in range(2)]
    xs = [d.x * (k + 1) + k for k in range(14)]
    want = []
    for x in xs:
        B.csr5_spmv_ex(h, x, d.y)
        want.append(d.y.clone())
    torch.cuda.synchronize()
    graphs, captured = [], [torch.full_like(d.y, float("nan")) for _ in side]
    for x, y in zip(xs[12:], captured):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            B.csr5_spmv_ex(h, x, y)
    alone = []
    for graph, y in zip(graphs, captured):
        graph.replay()
        torch.cuda.synchronize()
        alone.append(y.clone())
    for call in range(4):
        ys = [torch.full_like(d.y, float("nan")) for _ in streams * 2]
        for y in captured:
            y.fill_(float("nan"))
        torch.cuda.synchronize()
        for k, (x, y) in enumerate(zip(xs, ys)):
            if k % 3 == 0:
                with torch.cuda.stream(side[k // 3 % 2]):
                    graphs[k // 3 % 2].replay()
            B.csr5_spmv_ex(h, x, y, stream=streams[k % 6])
        torch.cuda.synchronize()
        for k, (y, w) in enumerate(zip(ys, want)):
            assert torch.equal(y[:fixed], w[:fixed]), (call, k)
        for k, (y, w) in enumerate(zip(captured, alone)):
            assert torch.equal(y[:fixed], w[:fixed]), (call, "replay", k)
    bar = 2e-12 * oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, xs[12].cpu().numpy())[1] + 1e-300
    assert np.all(np.abs((alone[0] - want[12]).cpu().numpy()) <= bar)
    B.csr5_free(h)


def test_nan_and_infinities_of_x_reach_their_rows_only():
    a = _far(1_100_001, 200 * BLOCK + 1, 15, 25, 0.1, seed=4)
    d = DeviceCsr(a)
    h = convert(d, use_workspace=False)
    assert B.csr5_get_form(h)["kernel"] == B.CSR5_KERNEL_GATHERED
    x = a.x.copy()
    x[[0, BLOCK - 1, BLOCK, 200 * BLOCK]] = [np.nan, np.inf, -np.inf, np.nan]
    d.x = torch.from_numpy(x).cuda()
    B.csr5_spmv_ex(h, d.x, d.y)
    torch.cuda.synchronize()
    y, (want, s) = d.y.cpu().numpy(), oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, x)
    odd = ~np.isfinite(want)
    assert 0 < odd.sum() < a.m and np.array_equal(np.isnan(y), np.isnan(want)) and np.array_equal(y[odd & ~np.isnan(want)], want[odd & ~np.isnan(want)])
    assert np.all(np.abs(y[~odd] - want[~odd]) <= 1e-12 * s[~odd] + 1e-300)
    B.csr5_free(h)


@pytest.mark.parametrize("m,n,how", [(1_100_000, 200 * BLOCK, "workspace"), (1_100_000, 200 * BLOCK, "not waited for"), (1_100_000, 200 * BLOCK, "two kernels"),
                                     (1_100_000, 200_000, "small x"), (1_100_000, 1024 * BLOCK + 1, "largest x"), (600_000, 200 * BLOCK, "few entries")])
def test_left_alone(m, n, how):
    """What a conversion that enqueues only, brings its memory or fixes the form gets, x that caches hold or that has too many
    blocks, and entries that would not pay for the lists in four products."""
    a = _far(m, n, 15, 25, 0.0, seed=2)
    d = DeviceCsr(a)
    flags = {"not waited for": B.CSR5_FLAG_NO_HOST_CHECK, "two kernels": B.CSR5_FLAG_AUX_TWO_KERNELS}.get(how, B.CSR5_FLAG_NONE)
    h = convert(d, use_workspace=how == "workspace", flags=flags)
    assert B.csr5_get_form(h)["kernel"] != B.CSR5_KERNEL_GATHERED
    check_spmv(d, h, how)
    B.csr5_free(h)


def test_columns_that_few_lines_hold_are_left_alone():
    """Power-law columns in random order, a band too wide for a window, rows as long as several tiles."""
    g = np.random.default_rng(7)
    for kind in ("power law", "band", "long rows"):
        n = 200 * BLOCK
        m, length = (9000, 2400) if kind == "long rows" else (1_100_000, 20)
        rows = np.repeat(np.arange(m, dtype=np.int64), length)
        if kind == "power law":
            col = g.permutation(n)[np.minimum(g.zipf(1.5, rows.size) - 1, n - 1)]
        elif kind == "band":
            col = (rows * n // m + g.integers(-100_000, 100_001, rows.size)).clip(0, n - 1)
        else:
            col = g.integers(0, n, rows.size)
        col = (np.sort(rows * n + col) - rows * n).astype(np.int32)
        a = wl.Csr(m=m, n=n, row_ptr=np.arange(0, m * length + 1, length, dtype=np.int32), col_idx=col, val=g.uniform(-1, 1, rows.size),
                   x=g.uniform(-1, 1, n), name=kind)
        d = DeviceCsr(a)
        h = convert(d, use_workspace=False)
        assert B.csr5_get_form(h)["kernel"] != B.CSR5_KERNEL_GATHERED, kind
        check_spmv(d, h, kind)
        B.csr5_free(h)
