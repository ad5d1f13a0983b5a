"""A propagator line pass gives the same bits wherever its cells lie in memory:
lines at offsets of up to a cache line in and out, and a batch of segments at
offsets that differ from one run to the next."""
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


@pytest.mark.parametrize("bc", [PER, ZERO])
@pytest.mark.parametrize("n,steps", [(2048, 100), (20011, 80), (20012, 200), (2000003, 50)])
def test_line(ctx, bc, n, steps):
    u0 = workloads.uniform(n, 990, steps, -1, 1, np.float32)
    first = None
    for si, so in ((0, 0), (0, 1), (3, 2), (5, 31), (0, 16), (2, 3)):
        src = upload(ctx, np.concatenate([np.zeros(si, np.float32), u0]))
        out = upload(ctx, np.full(n + so + 64, 7.0, np.float32))
        run(ctx, hx.stencil_args(dims=1, dtype=hx.HX_F32, nx=n, steps=steps, r=0.2, inp=src, out=out,
                                 in_offset=4 * si, out_offset=4 * so, bc_lo=bc, bc_hi=bc,
                                 time_block=steps))
        res = download(ctx, out, n + so + 64, np.float32)
        for b in (src, out):
            hx.hx_buffer_destroy(ctx, b)
        assert np.all(res[:so] == 7.0) and np.all(res[so + n:] == 7.0)
        first = res[so:so + n] if first is None else first
        assert np.array_equal(res[so:so + n], first), (si, so)


def test_batch(ctx):
    sizes = [250000 + 1000 * k for k in range(16)] + [257, 1024, 4095, 4097]
    rates = np.random.default_rng(1).uniform(0.05, 0.25, len(sizes))
    data = [workloads.uniform(m, 991, k, 0, 1, np.float32) for k, m in enumerate(sizes)]
    first = None
    for gap in (0, 1, 7, 33):
        off = np.cumsum([gap] + [m + gap for m in sizes])
        u0 = np.zeros(off[-1], np.float32)
        for o, x in zip(off, data):
            u0[o:o + x.size] = x
        src, out = upload(ctx, u0), hx.hx_buffer_create(ctx, u0.nbytes)
        segs = [hx.segment(inp=src, in_offset=4 * int(o), out=out, out_offset=4 * int(o), n=m,
                           r=float(r), bc_lo=PER, bc_hi=PER)
                for o, m, r in zip(off, sizes, rates)]
        plan = hx.hx_plan_create_batched(ctx, hx.HX_F32, 40, segs, form=hx.HX_FORM_AUTO)
        ev = hx.hx_launch_batched(ctx, plan)
        assert hx.hx_wait(ctx, ev) == hx.HX_OK, hx.hx_last_error(ctx)
        hx.hx_event_release(ctx, ev)
        got = download(ctx, out, u0.size, np.float32)
        hx.hx_plan_destroy(ctx, plan)
        for b in (src, out):
            hx.hx_buffer_destroy(ctx, b)
        res = [got[o:o + m] for o, m in zip(off, sizes)]
        first = first or res
        for k, (x, y) in enumerate(zip(res, first)):
            assert np.array_equal(x, y), (gap, k)
