"""GPU parity of the single-precision tile kernel that gathers neighbouring columns two at a time: the same bits as
the kernel that gathers them one by one (what a conversion that only enqueues gets), for runs of columns that begin
at even and odd places, cross rows and reach the last column, both tile heights, views at odd addresses; values
of x beside the ones asked for; and which columns are left alone."""
import pytest
import torch

from paper_1503_05032_amd import binding as B

pytestmark = pytest.mark.gpu


def _rows(m, n, starts, length, drop=0.0, seed=0):
    """m rows of runs of `length` columns that begin at the diagonal's place plus each of `starts`, clipped to the
    matrix; a share `drop` of the entries left out (runs of every length and place)."""
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    place = torch.arange(m, device="cuda:0") * n // m
    col = (place[:, None, None] + torch.tensor(starts, device="cuda:0")[None, :, None] + torch.arange(length, device="cuda:0")).view(m, -1)
    keep = (col >= 0) & (col < n) & (torch.rand(col.shape, generator=g, device="cuda:0") >= drop)
    keep[0, 0] = keep[-1, -1] = True
    col[0, 0], col[-1, -1] = 0, n - 1                            # the first and the last column
    row_ptr = torch.zeros(m + 1, dtype=torch.int32, device="cuda:0")
    row_ptr[1:] = torch.cumsum(keep.sum(1), 0)
    col = col[keep].int()
    val = torch.rand(col.numel(), generator=g, device="cuda:0") * 2 - 1
    x = torch.rand(n, generator=g, device="cuda:0") * 2 - 1
    return row_ptr, col, val, x


def _view(t, offset):
    whole = torch.empty(t.numel() + offset, dtype=t.dtype, device=t.device)
    whole[offset:] = t
    return whole[offset:]


def _product(m, n, row_ptr, col, val, x, sigma, flags, kernel):
    col, val = _view(col, col.data_ptr() // 4 % 4), val.clone()        # (the conversion reorders them)
    h = B.csr5s_convert_ex(m, n, col.numel(), row_ptr, col, val, sigma=sigma, flags=flags)
    assert B.csr5_get_form(h)["kernel"] == kernel, B.csr5_get_form(h)
    y = torch.full((m,), float("nan"), device="cuda:0")
    B.csr5s_spmv_ex(h, x, y)
    torch.cuda.synchronize()
    B.csr5_free(h)
    return y


@pytest.mark.parametrize("m,n,starts,length,drop,sigma,offset", [
    (400_000, 400_000, (-5000, -1, 3000), 3, 0.0, 0, 0), (300_001, 300_001, (-5000, -100, -1, 100, 3000), 3, 0.0, 0, 1),
    (1_000_003, 1_000_003, (-9000, -100, 0, 7000), 4, 0.05, 0, 3), (250_000, 500_001, (-40_000, -3000, 0, 3000), 6, 0.1, 0, 0),
    (900_000, 450_001, (-200, 0, 200), 5, 0.05, 16, 1), (400_000, 400_000, (-900, 0, 50, 1300, 9000, 20_000), 2, 0.0, 8, 0)])
def test_same_bits_as_one_by_one(m, n, starts, length, drop, sigma, offset):
    row_ptr, col, val, x = _rows(m, n, starts, length, drop, seed=m % 89)
    col, x = _view(col, offset), _view(x, offset)
    print("pairs", m, n, starts, length, drop, sigma, offset, col.numel(), flush=True)
    products = val.double() * x.double()[col.long()]
    want = torch.segment_reduce(products, "sum", offsets=row_ptr.long(), initial=0)
    scale = torch.segment_reduce(products.abs(), "sum", offsets=row_ptr.long(), initial=0)
    pairs = _product(m, n, row_ptr, col, val, x, sigma, B.CSR5_FLAG_NONE, B.CSR5_KERNEL_PAIRS)
    single = _product(m, n, row_ptr, col, val, x, sigma, B.CSR5_FLAG_NO_HOST_CHECK, B.CSR5_KERNEL_TILES)
    assert torch.equal(pairs, single)
    assert bool(((pairs.double() - want).abs() <= 1e-5 * scale + 1e-30).all())      # at most 64 additions per term: 64 * 2^-24 = 3.8e-6


def test_values_beside_the_ones_asked_for():
    """NaN in every column that no entry names: read along with its neighbour, and left out."""
    m = n = 600_000
    row_ptr, col, val, x = _rows(m, n, (-5000, -1, 3000), 6, 0.1, seed=1)
    named = torch.zeros(n, dtype=torch.bool, device="cuda:0")
    col = torch.where(col % 7 == 3, col - 1, col)                # (columns may repeat)
    named[col.long()] = True
    assert 0.1 < 1 - float(named.float().mean()) < 0.2
    x[~named] = float("nan")
    pairs = _product(m, n, row_ptr, col, val, x, 0, B.CSR5_FLAG_NONE, B.CSR5_KERNEL_PAIRS)
    assert bool(torch.isfinite(pairs).all())
    assert torch.equal(pairs, _product(m, n, row_ptr, col, val, x, 0, B.CSR5_FLAG_NO_HOST_CHECK, B.CSR5_KERNEL_TILES))


@pytest.mark.parametrize("starts,length", [(range(-12_000, 12_000, 997), 1), ((-1,), 3), ((-2,), 5), ((-8,), 16)])
def test_left_alone(starts, length):
    """Diagonals one by one, and bands whose 64 entries lie on a line or two."""
    m = n = 1_200_000
    row_ptr, col, val, x = _rows(m, n, list(starts), length)
    want = _product(m, n, row_ptr, col, val, x, 0, B.CSR5_FLAG_NO_HOST_CHECK, B.CSR5_KERNEL_TILES)
    assert torch.equal(_product(m, n, row_ptr, col, val, x, 0, B.CSR5_FLAG_NONE, B.CSR5_KERNEL_TILES), want)
