"""GPU test of the sum over a tile's columns (64 lanes, summed in rows of 16): segments that
begin and end beside the rows' boundaries keep their values apart, non-finite ones too."""
import numpy as np
import pytest
import torch

from paper_1503_05032_amd import binding as B

pytestmark = pytest.mark.gpu

# columns of a tile that the rows of the matrix take, in turn: boundaries at 15, 16, 17, 31, 32, 33, 47, 48, 49 and
# segments over one, two, three and four rows of 16
SPANS = [15, 1, 1, 14, 1, 1, 14, 1, 1, 15,   16, 16, 16, 16,   17, 15, 32,   33, 31,   1, 63,   48, 16,   49, 15,   63, 1,   64]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("sigma,cut", [(8, 0), (8, 1), (8, 7), (16, 0), (16, 9), (20, 3), (40, 5)])
def test_non_finite_values_stay_in_their_row(sigma, cut, dtype):
    """Every row gathers one element of x only: a NaN or an infinity there must reach that row and no other."""
    rng = np.random.default_rng(sigma + cut)
    lens = np.array(SPANS, dtype=np.int64) * sigma
    lens[0] -= cut                                       # row starts `cut` entries off the columns' edges
    lens[-1] += cut
    m, nnz = len(lens), int(lens.sum())
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.repeat(np.arange(m), lens).astype(np.int32)
    val = rng.uniform(0.5, 1.0, nnz)
    dev = "cuda:0"
    d = dict(row_ptr=torch.from_numpy(row_ptr).to(dev), col_idx=torch.from_numpy(col).to(dev), val=torch.from_numpy(val).to(dev, dtype))
    x = torch.from_numpy(rng.uniform(0.5, 1.0, m)).to(dev, dtype)
    y = torch.empty(m, dtype=dtype, device=dev)
    convert, spmv = (B.csr5_convert_ex, B.csr5_spmv_ex) if dtype is torch.float64 else (B.csr5s_convert_ex, B.csr5s_spmv_ex)
    expect = np.add.reduceat(d["val"].double().cpu().numpy(), row_ptr[:-1]) * x.double().cpu().numpy()
    h = convert(m, m, nnz, d["row_ptr"], d["col_idx"], d["val"], sigma=sigma)
    spmv(h, x, y)
    good = y.clone()
    # positive terms: at most one rounding per addition and product, and no term passes through more than 64 of either
    eps = 64 * (2.0 ** -53 if dtype is torch.float64 else 2.0 ** -24)
    assert np.all(np.abs(good.double().cpu().numpy() - expect) <= eps * expect)
    for r in range(m):
        for poison in (float("nan"), float("inf"), float("-inf")):
            bad = x.clone()
            bad[r] = poison
            spmv(h, bad, y)
            same = y == good
            same[r] = bool(torch.isnan(y[r])) if poison != poison else bool(y[r] == poison)
            assert bool(same.all()), (r, poison, torch.nonzero(~same).flatten().tolist())
    B.csr5_free(h)


@pytest.mark.parametrize("offset", [0, 1, 4])
@pytest.mark.parametrize("nnz", [1024, 4096, 5 * 4096 + 77, 3 * 1024 + 1])
def test_single_precision_tile_loads(nnz, offset):
    """Single precision with the look-behind at 16 entries per column: col_idx 16-byte aligned and not, one and
    several workgroups, the last one partly filled, an incomplete tile."""
    rng = np.random.default_rng(nnz + offset)
    lens = rng.integers(0, 33, nnz)
    lens = lens[:int(np.searchsorted(np.cumsum(lens), nnz))]
    lens = np.append(lens, nnz - lens.sum())
    m, n = len(lens), 5000
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = rng.integers(0, n, nnz).astype(np.int32)
    dev = "cuda:0"
    whole = torch.zeros(nnz + offset, dtype=torch.int32, device=dev)
    whole[offset:] = torch.from_numpy(col).to(dev)
    val = torch.from_numpy(rng.uniform(-1, 1, nnz)).to(dev, torch.float32)
    x = torch.from_numpy(rng.uniform(-1, 1, n)).to(dev, torch.float32)
    y = torch.full((m,), float("nan"), dtype=torch.float32, device=dev)
    products = val.double().cpu().numpy() * x.double().cpu().numpy()[col]
    ref, s = (np.add.reduceat(np.append(p, 0.0), row_ptr[:-1]) * (lens > 0) for p in (products, np.abs(products)))
    h = B.csr5s_convert_ex(m, n, nnz, torch.from_numpy(row_ptr).to(dev), whole[offset:], val, sigma=16)
    B.csr5s_spmv_ex(h, x, y)
    # a term passes through 16 + 6 + 4 additions and its product at most, 2^-24 each
    assert np.all(np.abs(y.double().cpu().numpy() - ref) <= 32 * 2.0 ** -24 * s)
    B.csr5_free(h)
