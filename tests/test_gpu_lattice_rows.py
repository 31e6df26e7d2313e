"""Laying out a lattice's rows takes what the same rows take with no edge along an axis: the count of such
edges does not wait for one counter."""
import ctypes as C
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CREATE = "_ZN2rt12model_createEPKdlPKlPKilPKfS5_bP12ihipStream_tPP8rt_modeli"  # rt::model_create


def test_lattice_rows_time(rt):
    """128^3 face-connected cubes, rows in point order (no sort on the host): half a million waves of rows."""
    import torch
    n = 128
    i = np.arange(n**3).reshape(n, n, n)
    nb = np.full((n, n, n, 6), -1, np.int64)
    nb[1:, :, :, 0], nb[:, 1:, :, 1], nb[:, :, 1:, 2] = i[:-1], i[:, :-1], i[:, :, :-1]
    nb[:, :, :-1, 3], nb[:, :-1, :, 4], nb[:-1, :, :, 5] = i[:, :, 1:], i[:, 1:], i[1:]
    nb = nb.reshape(-1, 6)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum((nb >= 0).sum(1))])).cuda()
    idx = torch.from_numpy(nb[nb >= 0].astype(np.int32)).cuda()
    grid = np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.float64)
    rt.load()
    fn = C.CDLL(rt.binding.LIB_PATH)[CREATE]
    fn.restype = C.c_int32
    fn.argtypes = [C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_bool,
                   C.c_void_p, C.c_void_p, C.c_int32]
    times = []
    for jitter in (0.2, 0.0):
        pos = torch.from_numpy(grid + np.random.default_rng(1).uniform(-jitter, jitter, grid.shape)).cuda()
        best = np.inf
        for _ in range(8):
            h = C.c_void_p()
            torch.cuda.synchronize()
            t = time.perf_counter()
            assert fn(pos.data_ptr(), n**3, off.data_ptr(), idx.data_ptr(), idx.numel(), None, None, False, None,
                      C.byref(h), 0) == 0
            best = min(best, time.perf_counter() - t)
            rt.load().rt_model_destroy(h)
        times.append(best)
    print(f"jittered {times[0] * 1e3:.2f} ms, lattice {times[1] * 1e3:.2f} ms")
    assert times[1] < 1.5 * times[0]
