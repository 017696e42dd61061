"""What a user of libcsr5 has it do, as measurable cases.

Two kinds of work, through the calls that `paper_1503_05032_amd.binding` offers:

  op "spmv"   one y = A*x on a handle that the program keeps (the conversion is in `prepare`, by the plain call
              that allocates for itself), repeated as an iterative solver repeats it
  op "cycle"  CSR -> CSR5 conversion, `iters` SpMVs, CSR5 -> CSR, release: what a program pays whose matrix is
              assembled anew in CSR order for every outer step

Matrices are drawn on the GPU from a seed, with the shapes of this repository's workloads: `uniform` (few short rows,
some empty), `stencil27` (27-point stencil on a g^3 grid), `powerlaw` (row lengths Zipf 2, columns preferring low ids),
`lp_rect` (30 % empty rows, short rows, a few dense ones), `mixed` (banded rows and log-normal random ones), `dense`,
`rows` (rows of one length, random columns) and `huge_mixed` (64-bit indices, long banded rows).

dtype is "f64" or "f32"; index is "i32" or "i64" (64-bit row pointers, double precision only); `offset` is where
col_idx begins inside a larger array, in elements (0 or 1: a view that is not 16-byte aligned).
"""
import math

import numpy as np
import torch

from paper_1503_05032_amd import binding as B
from paper_1503_05032_amd import workloads_device

DEVICE = "cuda:0"
ZIPF_MAX_ROW = 200_000          # longest row of a powerlaw matrix
LP_DENSE_ROW = 20_000           # length of the dense rows of an lp_rect matrix


# ---------------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------------
def _case(kind, op="spmv", dtype="f64", index="i32", offset=0, **more):
    return dict(kind=kind, op=op, dtype=dtype, index=index, offset=offset, **more)


def listed():
    cases = {
        # the smallest call: a circuit-sized matrix inside a host loop, launch and latency
        "spmv_uniform_2k": _case("uniform", m=2000, max_len=20),
        # a dense block stored as CSR: few long rows
        "spmv_dense_2k": _case("dense", n=2000),
        # the regular case: a 3-D discretisation, in double and in single precision
        "spmv_stencil_100": _case("stencil27", g=100),
        "spmv_stencil_100_f32": _case("stencil27", g=100, dtype="f32"),
        # a graph: very uneven rows, columns that prefer low ids
        "spmv_powerlaw_2m": _case("powerlaw", m=2_000_000),
        # rectangular LP/circuit matrix: empty rows, short rows, dense rows, uniform random columns
        "spmv_lp_rect": _case("lp_rect", m=1_500_000, n=4_000_000),
        # a mesh with irregular long-range couplings, x far larger than the caches
        "spmv_mixed_8m": _case("mixed", m=8_000_000),
        # rows of a few hundred entries whose col_idx is a view into a larger array, odd sizes
        "spmv_rows_201": _case("rows", m=30_011, n=60_013, length=201, offset=1),
        # the largest call: 64-bit indices, long banded rows
        "spmv_huge_mixed_i64": _case("huge_mixed", scale=0.25, index="i64"),
        # conversion there and back with a caller's workspace, only enqueued: regular matrix
        "cycle_stencil_100": _case("stencil27", "cycle", g=100, workspace=True, check=False, iters=1),
        # the same on a graph, with the blocking check of the input
        "cycle_powerlaw_2m": _case("powerlaw", "cycle", m=2_000_000, workspace=True, check=True, iters=1),
        # a solver's outer step on a small grid: plain conversion, 50 iterations, back
        "cycle_stencil_40_x50": _case("stencil27", "cycle", g=40, workspace=False, check=True, iters=50),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["uniform", "stencil27", "stencil27", "powerlaw", "lp_rect", "mixed", "dense", "rows", "rows", "huge_mixed"])
    c = _case(kind)
    if kind == "uniform":
        c.update(m=_log_int(rng, 300, 60_000), max_len=rng.randint(4, 40))
    elif kind == "stencil27":
        c.update(g=_log_int(rng, 16, 150))
    elif kind == "powerlaw":
        c.update(m=_log_int(rng, 20_000, 3_000_000))
    elif kind == "lp_rect":
        m = _log_int(rng, 20_000, 1_500_000)
        c.update(m=m, n=int(m * rng.uniform(1.0, 3.0)))
    elif kind == "mixed":
        c.update(m=_log_int(rng, 50_000, 5_000_000))
    elif kind == "dense":
        c.update(n=_log_int(rng, 150, 4000))
    elif kind == "rows":
        length = _log_int(rng, 5, 2000)
        c.update(m=max(3, _log_int(rng, 100_000, 30_000_000) // length), n=_log_int(rng, 8000, 400_000), length=length)
    else:
        c.update(scale=round(math.exp(rng.uniform(math.log(0.004), math.log(0.12))), 4), index="i64")
    if c["index"] == "i32":
        c["dtype"] = rng.choice(["f64", "f64", "f32"])
    c["offset"] = rng.choice([0, 0, 0, 1])
    if rng.random() < 0.3 and c["index"] == "i32":
        nnz = _expected(c)[2]                    # few iterations on the large ones: a pass stays short
        c.update(op="cycle", workspace=rng.random() < 0.7, check=rng.random() < 0.7,
                 iters=rng.choice([1, 1, 10, 50] if nnz < 2e6 else [1, 1, 5] if nnz < 2e7 else [1]))
    return c


# ---------------------------------------------------------------------------------------------------------------
# matrices, drawn on the GPU
# ---------------------------------------------------------------------------------------------------------------
def _running_max(t):
    """torch.cummax(t, 0).values of a long vector: blocks side by side, then the blocks' maxima."""
    block = 4096
    whole = torch.cat([t, t[-1:].expand(-t.numel() % block)]).view(-1, block)
    whole = torch.cummax(whole, 1).values
    before = torch.cummax(whole[:, -1], 0).values[:-1]
    whole[1:] = torch.maximum(whole[1:], before[:, None])
    return whole.view(-1)[:t.numel()]


def _from_lengths(lens, columns, n):
    """Columns of rows of the given lengths, sorted and distinct inside each row; `columns(rows, j)` draws the column
    of entry j of each row, and an entry that meets the one before it moves to the next free column."""
    rows = torch.repeat_interleave(torch.arange(lens.numel(), device=DEVICE), lens)
    j = torch.arange(rows.numel(), device=DEVICE) - (torch.cumsum(lens, 0) - lens)[rows]
    col = torch.sort(rows * n + columns(rows, j)).values - rows * n
    col = _running_max(rows * (2 * n) + col - j + n) - rows * (2 * n) - n + j
    return torch.minimum(col, n - lens[rows] + j).to(torch.int32)


def _rand(k, g):
    return torch.rand(k, generator=g, device=DEVICE, dtype=torch.float64)


def _zipf_distinct_tables():
    """Expected number of distinct columns below z (in units of the row's own scale) of a long stream of Zipf(1.5)
    draws: G(z) = integral of 1 - exp(-t^-1.5), as a table over log z."""
    z = np.exp(np.linspace(math.log(1e-4), math.log(1e9), 40_000))
    f = -np.expm1(-z ** -1.5)
    gz = z[0] + np.concatenate([[0.0], np.cumsum(0.5 * (f[1:] + f[:-1]) * np.diff(z))])
    return z, gz


def _interp(x, xp, fp):
    k = torch.searchsorted(xp, x).clamp_(1, xp.numel() - 1)
    x0, x1, f0, f1 = xp[k - 1], xp[k], fp[k - 1], fp[k]
    return f0 + (x - x0).clamp_(min=0) / (x1 - x0) * (f1 - f0)


def _powerlaw(m, fixed, g):
    n, longest = m, min(ZIPF_MAX_ROW, m)
    k = torch.arange(1, longest + 1, device=DEVICE, dtype=torch.float64)
    cdf = torch.cumsum(k ** -2.0, 0) / (math.pi ** 2 / 6)
    lens = (torch.searchsorted(cdf, _rand(m, fixed)) + 1).clamp_(max=longest)[torch.randperm(m, generator=g, device=DEVICE)]
    z, gz = (torch.from_numpy(t).to(DEVICE) for t in _zipf_distinct_tables())

    def columns(rows, j):                        # entry j of N: a random place in the j-th N-th of the distinct set
        want = lens[rows].double()
        scale = want / 2.679                     # G(infinity) = Gamma(1/3)
        part = (j.double() + _rand(j.numel(), g)) / want * _interp(n / scale, z, gz)
        return (_interp(part, gz, z) * scale).long().clamp_(0, n - 1)
    return lens, _from_lengths(lens, columns, n)


def _stencil27(grid):
    idx = torch.arange(grid ** 3, device=DEVICE)
    ix, iy, iz = idx % grid, (idx // grid) % grid, idx // (grid * grid)
    valid, offs = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                valid.append((ix + dx >= 0) & (ix + dx < grid) & (iy + dy >= 0) & (iy + dy < grid) & (iz + dz >= 0) & (iz + dz < grid))
                offs.append(dx + dy * grid + dz * grid * grid)
    valid = torch.stack(valid, 1)
    cols = (idx[:, None] + torch.tensor(offs, device=DEVICE)[None, :]).to(torch.int32)[valid]
    centre = (torch.tensor(offs, device=DEVICE) == 0).expand_as(valid)[valid]
    return valid.sum(1), cols, centre


def _matrix(c, seed):
    """dict(m, n, nnz, row_ptr, col, val, x) on the GPU; the values in double precision."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    kind = c["kind"]
    if kind == "huge_mixed":
        a = workloads_device.huge_mixed(DEVICE, scale=c["scale"], seed=seed)
        return dict(m=a["m"], n=a["n"], nnz=a["nnz"], row_ptr=a["row_ptr"], col=a["col_idx"], val=a["val"], x=a["x"])
    # Row lengths come in an order of the seed's, but are the same ones for every seed of a case: so is nnz.
    fixed = torch.Generator(device=DEVICE)
    fixed.manual_seed(20150503)
    lo, hi = -1.0, 1.0                           # values and x uniform in [lo, hi) unless said otherwise
    centre = None

    def anywhere(r, j):
        return torch.randint(0, n, r.shape, generator=g, device=DEVICE)
    if kind == "uniform":
        m = n = c["m"]
        lens = torch.randint(0, min(c["max_len"], n) + 1, (m,), generator=fixed, device=DEVICE)
        lens = lens[torch.randperm(m, generator=g, device=DEVICE)]
        col = _from_lengths(lens, anywhere, n)
    elif kind == "stencil27":
        m = n = c["g"] ** 3
        lens, col, centre = _stencil27(c["g"])
    elif kind == "powerlaw":
        m = n = c["m"]
        lo = 0.0
        lens, col = _powerlaw(m, fixed, g)
    elif kind == "lp_rect":
        m, n = c["m"], c["n"]
        u = _rand(m, fixed)
        lens = 1 + torch.floor(torch.log(1 - _rand(m, fixed)) / math.log(0.75)).long()
        lens[u < 0.3] = 0
        lens[u >= 0.999] = min(LP_DENSE_ROW, n // 4)
        lens = lens[torch.randperm(m, generator=g, device=DEVICE)]
        col = _from_lengths(lens, anywhere, n)
    elif kind == "mixed":
        m = n = c["m"]
        banded = _rand(m, fixed) < 0.8
        normal = torch.randn(m, generator=fixed, device=DEVICE, dtype=torch.float64)
        lens = torch.where(banded, torch.randint(8, 17, (m,), generator=fixed, device=DEVICE),
                           torch.exp(2.5 + 1.5 * normal).long().clamp_(1, n))
        order = torch.randperm(m, generator=g, device=DEVICE)
        banded, lens = banded[order], lens[order]

        def columns(r, j):
            near = (r + torch.randint(-5000, 5001, r.shape, generator=g, device=DEVICE)).clamp_(0, n - 1)
            return torch.where(banded[r], near, anywhere(r, j))
        col = _from_lengths(lens, columns, n)
    elif kind == "dense":
        m = n = c["n"]
        lens = torch.full((m,), n, device=DEVICE)
        col = torch.arange(n, device=DEVICE, dtype=torch.int32).repeat(m)
    elif kind == "rows":                         # one random column out of each `length`-th part of the columns
        m, n, length = c["m"], c["n"], min(c["length"], c["n"])
        lens = torch.full((m,), length, device=DEVICE)
        col = _from_lengths(lens, lambda r, j: ((j.double() + _rand(j.numel(), g)) * (n / length)).long().clamp_(max=n - 1), n)
    else:
        raise ValueError(kind)
    row_ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(lens, 0, out=row_ptr[1:])
    nnz = int(row_ptr[-1])
    if kind == "stencil27":                      # centre 26, neighbours -1 +- 0.01, x in [0, 1)
        val = -1.0 + (_rand(nnz, g) * 2 - 1) * 0.01
        val[centre] = 26.0
        x = _rand(n, g)
    elif kind == "lp_rect":                      # normal values
        val = torch.randn(nnz, generator=g, device=DEVICE, dtype=torch.float64)
        x = torch.randn(n, generator=g, device=DEVICE, dtype=torch.float64)
    else:
        val = lo + (hi - lo) * _rand(nnz, g)
        x = lo + (hi - lo) * _rand(n, g)
    return dict(m=m, n=n, nnz=nnz, row_ptr=row_ptr if c["index"] == "i64" else row_ptr.to(torch.int32), col=col, val=val, x=x)


# ---------------------------------------------------------------------------------------------------------------
# the program around the calls
# ---------------------------------------------------------------------------------------------------------------
class _Handle:
    """Keeps a conversion's handle and gives it back with the state."""

    def __init__(self, h):
        self.h = h

    def __del__(self):
        B.csr5_free(self.h, check=False)


def _calls(c):
    """(conversion, its workspace size, SpMV) of the case's types."""
    if c["index"] == "i64":
        return B.csr5l_convert_ex, B.csr5l_workspace_bytes, B.csr5_spmv_ex
    if c["dtype"] == "f32":
        return B.csr5s_convert_ex, B.csr5_workspace_bytes, B.csr5s_spmv_ex
    return B.csr5_convert_ex, B.csr5_workspace_bytes, B.csr5_spmv_ex


def prepare(case, seed):
    a = _matrix(case, seed)
    value = torch.float32 if case["dtype"] == "f32" else torch.float64
    val, x = a.pop("val").to(value), a.pop("x").to(value)
    col = a.pop("col")
    if case["offset"]:
        whole = torch.empty(col.numel() + case["offset"], dtype=torch.int32, device=DEVICE)
        whole[case["offset"]:] = col
        col = whole[case["offset"]:]
    y = torch.empty(a["m"], dtype=value, device=DEVICE)
    state = dict(a, case=case, val=val, col=col, x=x, y=y)
    convert, workspace_bytes, _ = _calls(case)
    if case["op"] == "cycle":
        state["ws"] = torch.empty(workspace_bytes(a["m"], a["nnz"]), dtype=torch.uint8, device=DEVICE) if case["workspace"] else None
        return state
    # a program that converts once: the plain call, which allocates for itself and checks its input
    if case["index"] == "i32" and case["dtype"] == "f64":
        h = B.csr5_convert(a["m"], a["n"], a["nnz"], a["row_ptr"], col, val)
    else:
        h = convert(a["m"], a["n"], a["nnz"], a["row_ptr"], col, val)
    state["handle"] = _Handle(h)
    state["call"] = B.csr5_spmv_bound(h, x, y)
    return state


def _view(ws, address, count, dtype):
    """`count` elements at a device address inside the workspace."""
    at = address - ws.data_ptr()
    return ws[at:at + count * dtype.itemsize].view(dtype)


def run(state):
    c = state["case"]
    if c["op"] == "spmv":
        state["call"]()
        return state["y"]
    convert, _, spmv = _calls(c)
    flags = B.CSR5_FLAG_NONE if c["check"] else B.CSR5_FLAG_NO_HOST_CHECK
    h = convert(state["m"], state["n"], state["nnz"], state["row_ptr"], state["col"], state["val"], workspace=state["ws"], flags=flags)
    for _ in range(c["iters"]):
        spmv(h, state["x"], state["y"])
    out = {"y": state["y"], "col": state["col"], "val": state["val"]}
    if state["ws"] is not None:                  # the format itself lies in the caller's workspace
        nnz, wide = state["nnz"], c["index"] == "i64"
        sigma = B.csr5_sigma_auto(nnz, state["m"])
        tile = 64 * sigma
        words = (sigma + 6 + (tile - 1).bit_length() + 31) // 32
        at = (B.csr5l_get_arrays if wide else B.csr5_get_arrays)(h)
        out["tile_ptr"] = _view(state["ws"], at["tile_ptr"], -(-nnz // tile) + 1, torch.int64 if wide else torch.int32)
        out["tile_desc"] = _view(state["ws"], at["tile_desc"], nnz // tile * words * 64, torch.int32)
    B.csr5_to_csr(h)
    B.csr5_free(h)
    return out


def exact(case, seed):
    a = _matrix(case, seed)
    if case["dtype"] == "f32":                   # the values the library is given
        a["val"], a["x"] = a["val"].float().double(), a["x"].float().double()
    products = a["val"] * a["x"][a["col"].long()]
    y = torch.segment_reduce(products, "sum", offsets=a["row_ptr"].long(), initial=0)
    if case["op"] == "spmv":
        return y
    out = {"y": y, "col": None, "val": a["val"]}   # back in CSR order
    if case["workspace"]:
        out.update(tile_ptr=None, tile_desc=None)
    return out


def _expected(c):
    """(m, n, nnz) of a case, nnz as its distribution gives it on average."""
    kind = c["kind"]
    if kind == "uniform":
        return c["m"], c["m"], c["m"] * c["max_len"] / 2
    if kind == "stencil27":
        return c["g"] ** 3, c["g"] ** 3, (3 * c["g"] - 2) ** 3
    if kind == "powerlaw":
        return c["m"], c["m"], c["m"] * (math.log(min(ZIPF_MAX_ROW, c["m"])) + 1.577) / (math.pi ** 2 / 6)
    if kind == "lp_rect":
        return c["m"], c["n"], c["m"] * (0.699 * 4 + 0.001 * min(LP_DENSE_ROW, c["n"] // 4))
    if kind == "mixed":
        return c["m"], c["m"], c["m"] * (0.8 * 12 + 0.2 * 37)
    if kind == "dense":
        return c["n"], c["n"], c["n"] ** 2
    if kind == "rows":
        return c["m"], c["n"], c["m"] * min(c["length"], c["n"])
    m = int(6_400_000 * c["scale"])
    return m, m, m * 0.97 * 359.5 + 5 * 0.47 * m


def work(case):
    m, n, nnz = _expected(case)
    v, i = (4 if case["dtype"] == "f32" else 8), (8 if case["index"] == "i64" else 4)
    spmv = nnz * (v + 4) + (n + m) * v + (m + 1) * i
    if case["op"] == "spmv":
        return {"bytes": spmv, "flops": 2 * nnz}
    # there and back: col_idx and val read and written twice; row_ptr read; the descriptors (a word per 16 entries) written
    convert = 4 * nnz * (v + 4) + (m + 1) * i + nnz / 4
    return {"bytes": convert + case["iters"] * spmv, "flops": 2 * nnz * case["iters"]}


def tolerance(case):
    # Another order of the sums (rows of up to hundreds of thousands of terms): measured against sums in 64 bits,
    # 4e-16 in double and 1.2e-7 in single precision over the listed cases and drawn ones; about four times that.
    # Indices, descriptors and values that only move stay the same ("differ" is 0).
    return {"rel": 5e-7, "max": 2e-5} if case["dtype"] == "f32" else {"rel": 2e-15, "max": 1e-13}
