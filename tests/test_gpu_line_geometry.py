"""1D runs whose geometry and pass depths are left to the library: any length,
step count, boundary and alignment against the oracle, and what needed a tmp
buffer or was refused before still does and is."""
import numpy as np
import pytest

import oracle
import workloads
from conftest import rel_l2

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, run, upload  # noqa: E402

TOL = {np.float64: 1e-12, np.float32: 1e-5}


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    hx.hx_tune_cache_clear()
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


def line(ctx, u0, r, steps, bc, shift=0, **kw):
    es = u0.itemsize
    bufs = [upload(ctx, np.concatenate([np.zeros(shift, u0.dtype), u0]))]
    bufs += [hx.hx_buffer_create(ctx, u0.nbytes + shift * es) for _ in range(2)]
    code = hx.HX_F64 if u0.dtype == np.float64 else hx.HX_F32
    off = dict(in_offset=shift * es, out_offset=shift * es, tmp_offset=shift * es)
    run(ctx, hx.stencil_args(dims=1, dtype=code, nx=u0.size, steps=steps, r=r, inp=bufs[0],
                             out=bufs[1], tmp=bufs[2], bc_lo=bc, bc_hi=bc, **off, **kw))
    res = download(ctx, bufs[1], u0.size, u0.dtype.type, offset=shift * es)
    for b in bufs:
        hx.hx_buffer_destroy(ctx, b)
    return res


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("bc", [hx.HX_BC_PERIODIC, hx.HX_BC_DIRICHLET0])
@pytest.mark.parametrize("n", [1, 3, 17, 411, 1000, 4099, 65537, 1 << 20, 3000001])
def test_library_choice(ctx, dtype, bc, n):
    u0 = workloads.uniform(n, 930, n % 1000, 0, 1, dtype)
    f = oracle.heat1d_periodic if bc == hx.HX_BC_PERIODIC else oracle.heat1d_dirichlet
    for steps, r in ((20, 0.25), (51, 0.05), (203, 0.2)):
        if n > 100000 and steps > 100:
            continue  # the oracle's time
        ref = f(u0.astype(np.float64), r, steps)
        if np.max(np.abs(ref)) < np.finfo(dtype).tiny:
            continue  # one cell between zero ends decays as 0.6^t: below the type's range
        got = line(ctx, u0, r, steps, bc, shift=steps % 4)
        assert rel_l2(got, ref) <= TOL[dtype], (steps, r)
        one = line(ctx, u0, r, steps, bc, time_block=steps)
        assert rel_l2(one, ref) <= TOL[dtype], (steps, r)


def test_tmp_and_refusals(ctx):
    n = 5000
    a, b = (hx.hx_buffer_create(ctx, n * 4) for _ in range(2))
    kw = dict(dims=1, dtype=hx.HX_F32, nx=n, r=0.25, inp=a, out=b)
    run(ctx, hx.stencil_args(steps=50, **kw))
    with pytest.raises(hx.HxError):
        hx.hx_launch_stencil(ctx, hx.stencil_args(steps=51, **kw))
    run(ctx, hx.stencil_args(steps=60, time_block=60, **kw))
    with pytest.raises(hx.HxError):  # beyond a tile of 32 cells per lane
        hx.hx_launch_stencil(ctx, hx.stencil_args(steps=1100, time_block=1100, **kw))
