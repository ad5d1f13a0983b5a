"""Non-finite cells near the ends of lines that the propagator pass advances:
infinite, negative infinite and NaN where the direct form has them (a zero end
is 0, not the sum of opposite cells), and finite everywhere else."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, run, upload  # noqa: E402

PER, ZERO = hx.HX_BC_PERIODIC, hx.HX_BC_DIRICHLET0


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    hx.hx_tune_cache_clear()
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


@pytest.mark.parametrize("bc", [ZERO, PER])
@pytest.mark.parametrize("n,steps", [(4096, 80), (20011, 80), (20011, 200), (8191, 256)])
def test_same_infinities_as_stepping(ctx, bc, n, steps):
    for at, value in ((0, np.inf), (1, -np.inf), (17, np.inf), (n - 1, -np.inf), (n - 3, np.inf),
                      (n - 40, np.nan), (n // 2, np.inf)):
        u0 = workloads.uniform(n, 960, at, 0, 1, np.float32)
        u0[at] = value
        src, out = upload(ctx, u0), hx.hx_buffer_create(ctx, u0.nbytes + 4)
        res = []
        for kw in (dict(), dict(cells_per_lane=16)):
            run(ctx, hx.stencil_args(dims=1, dtype=hx.HX_F32, nx=n, steps=steps, r=0.2, inp=src,
                                     out=out, out_offset=4, bc_lo=bc, bc_hi=bc, time_block=steps,
                                     **kw))
            res.append(download(ctx, out, n, np.float32, offset=4))
        for b in (src, out):
            hx.hx_buffer_destroy(ctx, b)
        got, want = res
        if n > 8000:  # this form, not the direct one (a shorter line is stepped in all blocks)
            assert not np.array_equal(got, want, equal_nan=True)
        fin = np.isfinite(want)
        assert not fin.all() and np.array_equal(got[~fin], want[~fin], equal_nan=True), at
        assert np.max(np.abs(got[fin] - want[fin])) <= 1e-5
