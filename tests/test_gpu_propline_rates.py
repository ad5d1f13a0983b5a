"""The propagator line pass on combs of lone values, over the rates it serves:
between two values an output consists of one or two taps' products, so an error
of a single small tap shows (in noise and smooth fields the large taps cover
it).  Each cell against the oracle, and the form's error against stepping's.

Tolerance of a cell, all cells positive: what the form omits is within 2^-21 of
an output by its accuracy check, the two-term splits of a cell and a tap add
3 2^-22, and the sums of a window's up to ten chunks, two accumulators, twenty
roundings of 2^-24 where every chunk contributes; a comb's outputs come from few
chunks: below 2^-19 together."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, run, upload  # noqa: E402

PER = hx.HX_BC_PERIODIC


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    hx.hx_tune_cache_clear()
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


@pytest.mark.parametrize("every", [3, 4, 5])
@pytest.mark.parametrize("r,D", [(0.0012, 27), (0.0015, 20), (0.004, 20), (0.01, 31), (0.03, 20),
                                 (0.05, 20), (0.13, 70), (0.25, 20)])
def test_combs(ctx, r, D, every):
    n = 1 << 22
    g = np.random.default_rng(every)
    u0 = np.zeros(n, np.float32)
    u0[::every] = 0.5 + 0.5 * g.random(u0[::every].size)
    src, out = upload(ctx, u0), hx.hx_buffer_create(ctx, u0.nbytes)
    ref = oracle.heat1d_periodic(u0.astype(np.float64), r, D)
    errs, res = [], []
    for kw in (dict(), dict(cells_per_lane=16)):
        run(ctx, hx.stencil_args(dims=1, dtype=hx.HX_F32, nx=n, steps=D, r=r, inp=src, out=out,
                                 bc_lo=PER, bc_hi=PER, time_block=D, **kw))
        res.append(download(ctx, out, n, np.float32))
        errs.append(np.abs(res[-1] - ref) / ref)
    for b in (src, out):
        hx.hx_buffer_destroy(ctx, b)
    if every == 3:  # this form, not the direct one (sparse combs at low rates are stepped)
        assert not np.array_equal(*res)
    print(f"r {r} D {D} every {every}: worst cell {errs[0].max():.2e} (stepping "
          f"{errs[1].max():.2e}), rms {np.sqrt((errs[0] ** 2).mean()):.2e} "
          f"({np.sqrt((errs[1] ** 2).mean()):.2e})")
    assert errs[0].max() <= 2.0 ** -19, int(np.argmax(errs[0]))
    assert (errs[0] ** 2).mean() <= (errs[1] ** 2).mean()
