"""Wrapping and releasing several regions in one call: the handles name the
regions, empty regions give no handle, and a handle that is gone is reported
after all others were released."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")


def test_wrap_many():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    ctx = hx.hx_ctx_create(0)
    raw = hx.hx_buffer_create(ctx, 4096)
    base, _ = hx.hx_buffer_ptr(ctx, raw)
    h = hx.hx_buffer_wrap_many(ctx, [(base, 256), (None, 0), (base + 256, 0), (base + 512, 1024)])
    assert h[1] == 0 and h[2] == 0 and 0 not in (h[0], h[3])
    assert hx.hx_buffer_ptr(ctx, h[0]) == (base, 256)
    assert hx.hx_buffer_ptr(ctx, h[3]) == (base + 512, 1024)
    hx.hx_buffer_destroy_many(ctx, h)
    again = hx.hx_buffer_wrap_many(ctx, [(base, 16)])
    both = (ctypes.c_uint64 * 2)(h[0], again[0])  # the first is gone
    with pytest.raises(Exception):
        hx.hx_buffer_destroy_many(ctx, both)
    with pytest.raises(Exception):
        hx.hx_buffer_ptr(ctx, again[0])  # released all the same
    assert len(hx.hx_buffer_wrap_many(ctx, [])) == 0
    hx.hx_buffer_destroy(ctx, raw)
    hx.hx_ctx_destroy(ctx)
