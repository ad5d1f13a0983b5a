"""Bands whose two ping-pong buffers are one buffer are refused, whatever form
the run takes (a pass reads rows after it has stored others), and nothing is
launched; a run of no steps leaves such buffers alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, upload  # noqa: E402

NX, ROWS = 64, [32, 40]


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


@pytest.mark.parametrize("mode,nodes", [(hx.HX_PART_GRAPH, False), (hx.HX_PART_GRAPH, True),
                                        (hx.HX_PART_BATCHED, False), (hx.HX_PART_BATCHED, True)])
def test_one_buffer_in_both_sets_is_refused(ctx, mode, nodes):
    u = [np.full((m, NX), 1.0 + k, np.float32) for k, m in enumerate(ROWS)]
    a = [upload(ctx, x) for x in u]
    b0 = hx.hx_buffer_create(ctx, u[0].nbytes)
    kw = dict(mode=mode, dims=2, nx=NX, periodic=False)
    with pytest.raises(hx.HxError, match="overlap"):
        hx.hx_run_partitioned(ctx, hx.partitioned_desc(hx.HX_F32, ROWS[1:], a[1:], a[1:], 8, 0.2,
                                                       **kw), node_events=nodes)
    if not nodes:  # (the node form finds the second band's after the first's launch)
        with pytest.raises(hx.HxError, match="overlap"):
            hx.hx_run_partitioned(ctx, hx.partitioned_desc(hx.HX_F32, ROWS, a, [b0, a[1]], 8, 0.2,
                                                           **kw), node_events=nodes)
    ev, in_b, _ = hx.hx_run_partitioned(ctx, hx.partitioned_desc(hx.HX_F32, ROWS, a, a, 0, 0.2,
                                                                 **kw), node_events=nodes)
    assert hx.hx_wait(ctx, ev) == hx.HX_OK and not in_b
    for x, y in zip(a, u):
        assert np.array_equal(download(ctx, x, y.shape, np.float32), y)
