"""Reverse sweeps of three and more streaming passes per segment (rows per block
given), whose middle passes add to the accumulator in place, on grids that end
one to three columns into a strip: the same bits as single steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from test_gpu_vc_ragged import gradient, stepped  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("nx", [248, 249, 250, 251, 252, 497, 747])
def test_middle_passes_add_once(ctx, dtype, nx):
    shape, T, S = (300, nx), 14, 14
    want = stepped(ctx, shape, dtype, T, S)
    for rows in (16, 7):
        for x, y in zip(gradient(ctx, shape, dtype, T, S, 0, rows), want):
            assert np.array_equal(x, y), rows
