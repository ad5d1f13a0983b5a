"""Runs of one checkpoint segment whose output is their input's buffer (uT = u0,
lam0 = lamT): the same bits as with two buffers, from two steps on, in whatever
passes the library takes."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, upload  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(64, 256), (300, 777), (9, 3)])
@pytest.mark.parametrize("rows", [0, 8])
def test_in_place(ctx, dtype, shape, rows):
    ny, nx = shape
    code = hx.HX_F64 if dtype == np.float64 else hx.HX_F32
    u0, kap = (workloads.uniform(shape, 970 + k, nx, 0.05, 1, dtype) for k in range(2))
    lam = workloads.uniform(shape, 972, nx, -1, 1, dtype)
    k = upload(ctx, kap)
    for T in (2, 3, 5, 8, 12, 13):
        res = []
        for same in (False, True):
            u, lT = upload(ctx, u0), upload(ctx, lam)
            uT = u if same else hx.hx_buffer_create(ctx, u0.nbytes)
            l0 = lT if same else hx.hx_buffer_create(ctx, u0.nbytes)
            u_again = upload(ctx, u0)
            bufs = [hx.hx_buffer_create(ctx, n * u0.nbytes) for n in (1, 2, max(T - 1, 1), 1)]
            ck, work, seg, gacc = bufs
            g = hx.hx_buffer_create(ctx, 8 * nx * ny)
            tail = (ck, work, seg, lT, l0, g, gacc, rows)
            e = hx.hx_heat_vc_forward(ctx, hx.hx_vc_args(code, nx, ny, 0.2, T, T, u, k, uT, *tail))
            e2 = hx.hx_heat_vc_backward(ctx, hx.hx_vc_args(code, nx, ny, 0.2, T, T, u_again, k, uT,
                                                           *tail), [e])
            assert hx.hx_wait(ctx, e2) == hx.HX_OK, hx.hx_last_error(ctx)
            res.append((download(ctx, uT, shape, dtype), download(ctx, l0, shape, dtype),
                        download(ctx, g, shape, np.float64)))
            for b in {u, uT, lT, l0, u_again, g, *bufs}:
                hx.hx_buffer_destroy(ctx, b)
        for x, y in zip(*res):
            assert np.array_equal(x, y), T
    hx.hx_buffer_destroy(ctx, k)
