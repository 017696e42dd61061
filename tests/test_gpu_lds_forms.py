"""What both SpMVs with x through LDS have to do beside the right sums: several products of one
handle in flight at once, matrices with columns out of range refused by a conversion that
samples them, and the largest number of rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_05032_amd import binding as B

from gpu_util import DeviceCsr, convert
from test_gpu_staged import _rows
from test_gpu_window import _band

pytestmark = pytest.mark.gpu

FORMS = [B.CSR5_KERNEL_PARTS, B.CSR5_KERNEL_WINDOW]


def _matrix(form):
    return _rows(30_011, 201, 60_013, seed=9, mixed=True) if form == B.CSR5_KERNEL_PARTS else _band(50_001, 90_003, 60, 110, 5000, 0.1, True, seed=9)


@pytest.mark.parametrize("form", FORMS)
def test_four_products_in_flight_on_two_streams(form):
    a = _matrix(form)
    d = DeviceCsr(a)
    h = convert(d)
    assert B.csr5_get_form(h)["kernel"] == form
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    rng = np.random.default_rng(3)
    xs = [rng.standard_normal(a.n) for _ in range(4)]
    xd = [torch.from_numpy(x).to("cuda:0") for x in xs]
    refs = [oracle.csr_spmv(a.m, a.row_ptr, a.col_idx, a.val, x) for x in xs]
    for rnd in range(5):
        ys = [torch.full_like(d.y, float("nan")) for _ in range(4)]
        torch.cuda.synchronize()
        for k in range(4):
            B.csr5_spmv_ex(h, xd[k], ys[k], stream=(s1, s2)[k % 2])
        s1.synchronize()
        s2.synchronize()
        for k, (want, s) in enumerate(refs):
            assert np.all(np.abs(ys[k].cpu().numpy()[:a.m] - want) <= 1e-12 * s + 1e-300), (rnd, k)
    B.csr5_free(h)


@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("form", FORMS)
def test_columns_out_of_range_are_refused(form, single):
    """One column in 97 is out of range, so that the samples meet some."""
    a = _matrix(form)
    a.col_idx[::97] = np.array([a.n, -1, 2**31 - 1, -2**31], dtype=np.int32)[np.arange(a.col_idx[::97].size) % 4]
    d = DeviceCsr(a)
    val = d.val.float() if single else d.val
    kept = val.clone()
    rc, h = (B.csr5s_convert_ex if single else B.csr5_convert_ex)(a.m, a.n, a.nnz, d.row_ptr, d.col_idx, val, check=False)
    assert rc == B.CSR5_EINVAL and not h
    torch.cuda.synchronize()
    assert np.array_equal(d.col_idx.cpu().numpy(), a.col_idx) and torch.equal(val, kept)


@pytest.mark.parametrize("form,length,n", [(B.CSR5_KERNEL_PARTS, 201, 60_013), (B.CSR5_KERNEL_WINDOW, 12, 300_000)])
def test_largest_row_count(form, length, n):
    """2^31 - 2 rows, nearly all of them empty: the zeroes at the end of y, and nothing behind it."""
    free, _ = torch.cuda.mem_get_info()
    if free < 80 * 2**30:
        pytest.skip("needs about 60 GB of GPU memory")
    m, live, dev = 2**31 - 2, 6_000_000 // 201 if form == B.CSR5_KERNEL_PARTS else 300_000, torch.device("cuda:0")
    rows = torch.arange(live, device=dev, dtype=torch.int64) * (m - 1) // (live - 1)           # the first and the last among them
    row_ptr = torch.empty(m + 1, dtype=torch.int32, device=dev)
    for k in range(0, m + 1, 2**28):                                                          # row_ptr[r]: entries of the rows before r
        e = min(m + 1, k + 2**28)
        row_ptr[k:e] = torch.searchsorted(rows, torch.arange(k, e, device=dev, dtype=torch.int64)) * length
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    if form == B.CSR5_KERNEL_PARTS:
        col = torch.randint(0, n, (live, length), generator=g, device=dev)
    else:
        col = (torch.arange(live, device=dev)[:, None] * n // live + torch.randint(-5000, 5001, (live, length), generator=g, device=dev)).clamp_(0, n - 1)
    col = torch.sort(col, dim=1).values
    val, x = (torch.rand(k, generator=g, device=dev, dtype=torch.float64) * 2 - 1 for k in (live * length, n))
    products = val.view(live, length) * x[col]
    want, scale = products.sum(1), products.abs().sum(1)
    whole = torch.full((m + 4096,), 7.0, dtype=torch.float64, device=dev)
    y = whole[2048:2048 + m]
    entries = col.to(torch.int32).view(-1)
    h = B.csr5_convert_ex(m, n, live * length, row_ptr, entries, val, sigma=8)
    assert B.csr5_get_form(h)["kernel"] == form
    print("largest row count", form, live, flush=True)
    B.csr5_spmv_ex(h, x, y)
    torch.cuda.synchronize()
    assert bool(((y[rows] - want).abs() <= 1e-12 * scale + 1e-300).all())
    y[rows] = 0
    assert bool((whole[:2048] == 7).all()) and bool((whole[2048 + m:] == 7).all())
    for k in range(0, m, 2**28):
        assert not bool(y[k:k + 2**28].any()), k
    B.csr5_free(h)
