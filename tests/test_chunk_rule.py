"""The chunk length of one-step 3D launches: the measured best lengths, and chunks
that with their halo stay below the 2 GiB a buffer can address, down to the
grids that plan creation refuses.  Host only."""
import ctypes

import numpy as np
import pytest

from paper_2211_06300_amd import esi


def _chunk(nxp, nyp, nzp, ns, plane=None):
    f = esi.load_library().esi_host_step3d_chunk
    f.restype = ctypes.c_int
    if plane is None:
        xs = -(-(-(-nxp // 64) * 64 + 16) // 32) * 32
        plane = xs * (-(-nyp // 16) * 16 + 16)
    return f(nxp, nyp, nzp, ctypes.c_int64(plane), ns)


@pytest.mark.parametrize("n,ns,planes", [(40, 1, 4), (48, 1, 5), (64, 1, 3), (64, 2, 6), (96, 1, 8), (163, 1, 7), (256, 4, 8)])
def test_measured_lengths(n, ns, planes):
    assert _chunk(n + 40, n + 40, n + 40, ns) == planes


def test_every_length_is_taken():
    # padded 64 x 16 x (nz + 8) grids
    cases = [(17, 20), (17, 29), (17, 37), (21, 86), (17, 57), (21, 103)]
    assert [_chunk(64, 16, nz + 8, ns) for nz, ns in cases] == [3, 4, 5, 6, 7, 8]


@pytest.mark.parametrize("planes", range(1, 9))
def test_a_chunk_fits_its_buffer(planes):
    most = (2 ** 31 - 1) // (4 * (planes + 9))      # largest plane for `planes` and their halo
    for plane in (most, most + 1):
        ch = _chunk(6000, 6000, 40, 1, plane)
        assert ch == 0 or (ch + 9) * 4 * plane < 2 ** 31
        assert (ch >= 1) == (10 * 4 * plane < 2 ** 31)
        assert ch <= planes if plane == most and planes < 8 else True
        assert ch < planes if plane == most + 1 else ch >= min(planes, 3)


def test_a_plane_too_large_is_refused():
    lib = esi.load_library()
    src, ptr = np.zeros((1, 3), np.int32), np.zeros(2, np.int64)
    geo = esi._Geom(1, src.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)),
                    ptr.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), None)
    grid = esi._Grid(3, 1, 7400, 7400, 4, 10, 10.0, 1e-3, -1.0, 0.0, 1.0)
    h = ctypes.c_void_p()
    fake = ctypes.c_void_p(16)   # never dereferenced
    assert lib.esi_plan_create(ctypes.byref(h), ctypes.byref(grid), ctypes.byref(geo), fake, None) == 2
    assert b"plane" in lib.esi_last_error()
