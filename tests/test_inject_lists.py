"""The receiver whose data a two-step 2D launch reads ahead for an injection
entry lies in the entry's own shot, also where cells hold several receivers and
a shot with fewer receivers follows: no address the launch forms leaves the
injected data.  Host only: the lists are built as a plan builds them."""
import ctypes

import numpy as np
import pytest

from paper_2211_06300_amd import esi


def _entries(nx, nz, nb, src, ptr, rec, rows):
    lib = esi.load_library()
    f = lib.esi_host_injection
    f.restype = ctypes.c_int64
    i32, i64 = ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int64)
    grid = esi._Grid(2, nz, nx, 1, nb, 4, 10.0, 1e-3, -1.0, 0.0, 1.0)
    src, ptr, rec = (np.ascontiguousarray(a, t) for a, t in ((src, np.int32), (ptr, np.int64), (rec, np.int32)))
    geo = esi._Geom(len(src), src.ctypes.data_as(i32), ptr.ctypes.data_as(i64), rec.ctypes.data_as(i32))
    n = f(ctypes.byref(grid), ctypes.byref(geo), rows, ctypes.c_int64(0), None)
    out = np.empty((n, 6), np.int32)
    assert f(ctypes.byref(grid), ctypes.byref(geo), rows, ctypes.c_int64(n), out.ctypes.data_as(i32)) == n
    return out


@pytest.mark.parametrize("rows", [8, 16, 24, 32, 40])
@pytest.mark.parametrize("nx,nz,nb", [(152, 88, 8), (37, 70, 4)])
def test_receiver_read_ahead_stays_in_its_shot(nx, nz, nb, rows):
    line = np.stack([np.arange(nx), np.full(nx, 3)], 1)
    gx, gz = np.meshgrid(np.arange(8, 28), np.arange(30, 50))
    block = np.stack([gx.ravel(), gz.ravel()], 1)
    # cells of two and of many receivers, then smaller shots, one of one receiver, one of none
    shots = [np.concatenate([line, block, block[:90], np.repeat(block[:1], 7, 0)]), line, line[:0], line[:1], line[5:9]]
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in shots])])
    out = _entries(nx, nz, nb, np.zeros((len(shots), 2)), ptr, np.concatenate(shots), rows)
    shot, ahead, first, count = out[:, 0], out[:, 3], out[:, 4], out[:, 5]
    assert count.min() == 1 and count.max() == 9
    nrec = np.diff(ptr)
    assert (ahead >= 0).all() and (ahead < nrec[shot]).all()
    np.testing.assert_array_equal(ahead, first)
    # and every sample of the batch's last step lies inside the data
    nt = 13
    assert (nt * ptr[shot] + (nt - 1) * nrec[shot] + ahead).max() < nt * ptr[-1]
