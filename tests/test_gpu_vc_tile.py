"""Variable-coefficient gradients whose passes are left to the library (on these
small grids the tile form, up to 12 steps a pass) against the streaming passes
(taken where the rows per block are given): the same bits, whatever the grid,
alignment, segment length and remainder, forward, recompute and sweep."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from test_gpu_vc_ragged import gradient  # noqa: E402

# around the tile's output: 232 to 248 columns, 8 to 44 rows; one and many tiles
SHAPES = [(1, 4), (2, 6), (12, 5), (16, 232), (17, 233), (24, 240), (41, 241), (45, 247),
          (64, 256), (97, 500), (150, 333), (333, 150)]


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", SHAPES)
def test_tile_equals_streaming(ctx, dtype, shape):
    for T, S in ((1, 1), (2, 2), (13, 6), (30, 12), (26, 13), (29, 29), (20, 0)):
        want = gradient(ctx, shape, dtype, T, S, 0, 8)
        got = gradient(ctx, shape, dtype, T, S, T % 4, 0)
        for x, y in zip(got, want):
            assert np.array_equal(x, y), (T, S)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("rows", [0, 8])
def test_totals_start_at_zero(ctx, dtype, rows):
    """The FP64 total and the accumulator may hold anything beforehand, also on
    a second run over the same buffers."""
    from test_gpu_vc_ragged import Dev, fields
    shape, T, S = (40, 241), 13, 6
    want = gradient(ctx, shape, dtype, T, S, 0, rows)[2]
    u0, kap, lam = fields(shape, dtype)
    d = Dev(ctx, shape, dtype, 0)
    code = hx.HX_F64 if dtype == np.float64 else hx.HX_F32
    seg, nseg = hx.hx_vc_schedule(T, S)
    bad = np.full(shape, np.nan)
    a = hx.hx_vc_args(code, shape[1], shape[0], 0.2, T, S, d.new(1, u0), d.new(1, kap), d.new(1),
                      d.new(nseg - 1), d.new(2), d.new(seg - 1), d.new(1, lam), d.new(1),
                      d.new(1, bad, es=8), d.new(1, bad.astype(dtype)), rows)
    for _ in range(2):
        e = hx.hx_heat_vc_backward(ctx, a, [hx.hx_heat_vc_forward(ctx, a)])
        assert hx.hx_wait(ctx, e) == hx.HX_OK, hx.hx_last_error(ctx)
        assert np.array_equal(d.get(a.gk64, np.float64), want)
    d.close()
