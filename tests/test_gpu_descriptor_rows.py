"""GPU parity of the descriptors where the transposition forms them from a tile's range of
rows: ranges of one and of several wavefronts, and around the 4096 rows beyond which the
row starts are searched for (a run of empty rows inside a tile, on its boundary, before the
first nonzero, behind the last one)."""
import numpy as np
import pytest
import torch

from paper_1503_05032_amd import binding as B
from paper_1503_05032_amd import workloads as wl

from gpu_util import DeviceCsr, check_format, check_spmv, convert

pytestmark = pytest.mark.gpu


def _lens(T, run, where):
    """Three tiles and a bit of rows of 0 to 5 entries with `run` empty rows in one place."""
    rng = np.random.default_rng(run + T)
    lens = rng.integers(0, 6, size=T)
    lens = lens[np.cumsum(lens) <= 3 * T + T // 3]
    at = {"front": 0, "inside": int(np.searchsorted(np.cumsum(lens), T + T // 2)), "end": len(lens)}.get(where)
    if at is None:                                       # exactly where tile 1 begins
        at = int(np.searchsorted(np.cumsum(lens), T)) + 1
        lens[at - 1] -= int(np.cumsum(lens)[at - 1]) - T
    return np.insert(lens, at, np.zeros(run, dtype=lens.dtype))


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("sigma", [1, 8, 16, 24, 33, 48])
def test_runs_of_empty_rows(sigma, wide):
    T = 64 * sigma
    rows = T // 2                                        # about as many rows begin in a tile
    for where in ("front", "inside", "boundary", "end"):
        for run in (0, 62, 65, 4096 - rows - 1, 4096 - rows // 2, 4096, 4097, 70_000):
            if run < 0:
                continue
            a = wl.from_row_lengths(_lens(T, run, where), 300, seed=run, name=f"{where}{run}")
            print("rows", sigma, wide, where, run, a.m, a.nnz, flush=True)
            d = DeviceCsr(a, wide=wide)
            h = convert(d, sigma=sigma)
            check_format(d, h, (a.name, sigma))
            check_spmv(d, h, (a.name, sigma))
            B.csr5_free(h)


@pytest.mark.parametrize("sigma", [8, 16])
def test_exact_range_limits(sigma):
    """Complete tiles whose ranges have 4095, 4096, 4097 rows: one entry per row but for one long first row."""
    T = 64 * sigma
    for span in (4095, 4096, 4097):
        tile = np.concatenate([[T - 10], np.zeros(span - 10, dtype=np.int64), np.ones(10, dtype=np.int64)])
        a = wl.from_row_lengths(np.tile(tile, 3), T + 50, seed=span, name=f"span{span}")
        assert a.nnz == 3 * T
        d = DeviceCsr(a)
        h = convert(d, sigma=sigma)
        check_format(d, h, (a.name, sigma))
        check_spmv(d, h, (a.name, sigma))
        B.csr5_to_csr(h)
        torch.cuda.synchronize()
        assert np.array_equal(d.col_idx.cpu().numpy(), a.col_idx)
        B.csr5_free(h)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("sigma", [1, 8, 16, 24, 48])
def test_rows_per_tile(sigma, wide):
    """Tiles in which exactly so many rows begin: a row per lane, one more, and the steps of four more per lane."""
    T = 64 * sigma
    for rows in (1, 63, 64, 65, 128, 129, 319, 320, 321, 577, T - 1, T):
        if rows > T:
            continue
        tile = np.concatenate([np.ones(rows - 1, dtype=np.int64), [T - rows + 1]])
        lens = np.concatenate([tile, tile, [0, 0], tile, tile[:rows // 2]])
        a = wl.from_row_lengths(lens, T + 50, seed=rows, name=f"rows{rows}")
        d = DeviceCsr(a, wide=wide)
        h = convert(d, sigma=sigma)
        check_format(d, h, (a.name, sigma))
        check_spmv(d, h, (a.name, sigma))
        B.csr5_free(h)
