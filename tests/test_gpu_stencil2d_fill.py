"""The deep float passes of the 2D band kernel in both forms of the pipeline's
fill (many waves: short chunks; few: tall ones): the same bits, on aligned and
ragged rows, whole and between halo rows, and the oracle's values."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, run, upload  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


@pytest.mark.parametrize("D", [10, 12, 16])
@pytest.mark.parametrize("ny,nx", [(1537, 2048), (1500, 2051)])
@pytest.mark.parametrize("r", [0.2, 0.24])
@pytest.mark.parametrize("ghost", [False, True])
def test_fills_agree(ctx, D, ny, nx, r, ghost):
    v0 = workloads.uniform((ny, nx), 995, D, 0, 1, np.float32)
    halo = workloads.uniform((2, D, nx), 996, D, 0, 1, np.float32)
    src, out = upload(ctx, v0), hx.hx_buffer_create(ctx, v0.nbytes)
    h = upload(ctx, halo)
    bc = hx.HX_BC_GHOST if ghost else hx.HX_BC_DIRICHLET0
    kw = dict(halo_lo=h, halo_hi=h, halo_hi_offset=4 * D * nx, halo_width=D) if ghost else {}
    res = []
    for rows in (256, 5, 1):  # 60 waves, over 3000, over 13000
        run(ctx, hx.stencil_args(dims=2, dtype=hx.HX_F32, nx=nx, ny=ny, steps=D, r=r, inp=src,
                                 out=out, bc_lo=bc, bc_hi=bc, time_block=D, rows_per_block=rows,
                                 cells_per_lane=4, waves_per_group=4, **kw))
        res.append(download(ctx, out, (ny, nx), np.float32))
    for b in (src, out, h):
        hx.hx_buffer_destroy(ctx, b)
    assert np.array_equal(res[0], res[1]) and np.array_equal(res[0], res[2])
    ext = np.concatenate([halo[0], v0, halo[1]]) if ghost else v0
    at = D if ghost else 0
    ref = oracle.heat2d_dirichlet(ext.astype(np.float64), r, D)[at:at + ny]
    assert np.max(np.abs(res[0] - ref)) <= 4 * D * 2.0 ** -24
