"""exp formed several at a time with its tables in a copy (cr_exp_n) gives the
bits of cr_exp for every argument: ordinary ones, those the first evaluation
cannot decide, the ends of the range, overflow, subnormal results and NaN."""
import ctypes as C

import numpy as np
import pytest


def _arguments():
    rng = np.random.default_rng(51)
    edge = np.array([0.0, -0.0, 709.7, 709.69999, -708.3, -708.29999, 709.79, -745.2, -720.0,
                     1e308, -1e308, np.inf, -np.inf, np.nan, 1e-300, np.log(2.0)])
    x = np.concatenate([rng.uniform(-45, 45, 200_000), rng.uniform(-750, 720, 50_000),
                        rng.uniform(-1e-5, 1e-5, 20_000), edge])
    return x, rng.permutation(x)


def test_host():
    from paper_1611_02274_amd import _lib
    f = _lib.lib().rkmi_crmath_host
    f.argtypes = [C.c_int, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p]
    x, y = _arguments()
    got = {}
    for fn in (0, 8, 9):
        got[fn] = np.empty_like(x)
        assert f(fn, x.size, x.ctypes.data, y.ctypes.data, got[fn].ctypes.data) == 0
    ey = np.empty_like(x)
    assert f(0, x.size, y.ctypes.data, x.ctypes.data, ey.ctypes.data) == 0
    for a, b in ((got[8], got[0]), (got[9], ey)):
        nan = np.isnan(b)
        assert np.array_equal(np.isnan(a), nan)
        assert np.array_equal(a[~nan].view(np.int64), b[~nan].view(np.int64))


@pytest.mark.gpu
def test_device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_02274_amd import _lib
    L = _lib.lib()
    fd, fh = L.rkmi_crmath_device, L.rkmi_crmath_host
    fd.argtypes = [C.c_int, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p]
    fh.argtypes = [C.c_int, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p]
    x, y = _arguments()
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    for fn in (8, 9):
        od = torch.empty_like(xd)
        assert fd(fn, x.size, xd.data_ptr(), yd.data_ptr(), od.data_ptr(), None) == 0
        torch.cuda.synchronize()
        want, got = np.empty_like(x), od.cpu().numpy()
        assert fh(fn, x.size, x.ctypes.data, y.ctypes.data, want.ctypes.data) == 0
        nan = np.isnan(want)
        assert np.array_equal(np.isnan(got), nan)
        assert np.array_equal(got[~nan].view(np.int64), want[~nan].view(np.int64))
