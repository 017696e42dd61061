"""What a conversion that is waited for learns from the device: many threads at a time, each on a stream of its own and
with a matrix of its own, good ones and bad ones; a conversion behind long work; the verdict after an error that the
caller's own HIP call left behind."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from paper_1503_05032_amd import binding as B

pytestmark = pytest.mark.gpu


def _matrix(seed):
    rng = np.random.default_rng(seed)
    m, n = int(rng.integers(300, 3000)), int(rng.integers(100, 5000))
    lens = rng.integers(1, 30, size=m)
    row_ptr = np.zeros(m + 1, dtype=np.int32)
    np.cumsum(lens, out=row_ptr[1:])
    col = rng.integers(0, n, size=row_ptr[-1]).astype(np.int32)
    if seed % 3 == 1:
        col[int(rng.integers(0, col.size))] = n                  # out of range
    if seed % 3 == 2:
        row_ptr[m // 2] += 40                                    # decreasing behind it
    return m, n, row_ptr, col


def test_many_threads():
    found, failed = {}, []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            for seed in range(5 * k, 5 * k + 5):
                m, n, row_ptr, col = _matrix(seed)
                with torch.cuda.stream(stream):
                    rp, c, v = (torch.from_numpy(t).cuda() for t in (row_ptr, col, np.ones(col.size)))
                    stream.synchronize()
                    try:
                        h = B.csr5_convert_ex(m, n, col.size, rp, c, v, stream=stream)
                        assert B.csr5_status(h) & 3 == 0
                        B.csr5_free(h)
                        found[seed] = True
                    except B.Csr5Error:
                        found[seed] = np.array_equal(c.cpu().numpy(), col) and None
        except Exception as e:                                   # (a thread's exception would only be printed)
            failed.append(e)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(40)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed[0]
    assert found == {seed: True if seed % 3 == 0 else None for seed in range(200)}


def test_behind_long_work():
    """Milliseconds of products that the conversion waits for."""
    m, n, row_ptr, col = _matrix(0)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        rp, c, v = (torch.from_numpy(t).cuda() for t in (row_ptr, col, np.ones(col.size)))
        a = torch.rand(8192, 8192, device="cuda:0")
        a @ a
        stream.synchronize()
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(4):
            a = a @ a
            a /= a.max()
        end.record()
        h = B.csr5_convert_ex(m, n, col.size, rp, c, v, stream=stream)
        assert end.query() and begin.elapsed_time(end) > 4
        assert B.csr5_status(h) & 3 == 0
        y, x = torch.empty(m, dtype=torch.float64, device="cuda:0"), torch.ones(n, dtype=torch.float64, device="cuda:0")
        B.csr5_spmv_ex(h, x, y, stream=stream)
        stream.synchronize()
        assert np.array_equal(y.cpu().numpy(), np.diff(row_ptr).astype(np.float64))
        B.csr5_free(h)


def test_status_beside_an_error_of_the_caller():
    """A call of the program's own that failed on this thread (a device that does not exist) is not the library's error."""
    m, n, row_ptr, col = _matrix(0)
    rp, c, v = (torch.from_numpy(t).cuda() for t in (row_ptr, col, np.ones(col.size)))
    h = B.csr5_convert_ex(m, n, col.size, rp, c, v)
    hip = ctypes.CDLL(B.LIB_PATH)                                # (the HIP runtime that the library is linked to)
    try:
        for _ in range(40):
            assert hip.hipSetDevice(1 << 20) != 0
            assert B.csr5_status(h) & 3 == 0
    finally:
        hip.hipGetLastError()
        B.csr5_free(h)
