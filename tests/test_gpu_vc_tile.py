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
