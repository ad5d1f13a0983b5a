"""The 2D pass in its two forms.  With the geometry left to the library small
grids take the tile form; a given rows_per_block takes the streaming form.  A
pass of one depth has the same bits in both, for every row length (also those
that are no multiple of the vector width) and row alignment; deep passes hold
the oracle's tolerance."""
import numpy as np
import pytest

import oracle
import workloads
from conftest import rel_l2

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, run, upload  # noqa: E402

TOL = {np.float64: 1e-12, np.float32: 1e-5}
# around the tile's 256 columns and 32 and 64 rows, and the smallest grids
SHAPES = [(1, 1), (2, 3), (5, 2), (31, 255), (32, 256), (33, 257), (64, 240), (65, 511),
          (130, 1023), (9, 700)]


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


def grid(ctx, u0, r, steps, shift=0, halo=None, **geom):
    """One run; `shift` cells in front of every operand move its rows off 16 bytes."""
    ny, nx = u0.shape
    dt = u0.dtype.type
    es = u0.itemsize
    pad = np.zeros(shift, dtype=dt)
    bi = upload(ctx, np.concatenate([pad, u0.ravel()]))
    bo, bt = (hx.hx_buffer_create(ctx, u0.nbytes + shift * es) for _ in range(2))
    kw = dict(bc_lo=hx.HX_BC_DIRICHLET0, bc_hi=hx.HX_BC_DIRICHLET0)
    bufs = [bi, bo, bt]
    if halo is not None:
        top, bot = (upload(ctx, np.concatenate([pad, h.ravel()])) for h in halo)
        bufs += [top, bot]
        kw = dict(bc_lo=hx.HX_BC_GHOST, bc_hi=hx.HX_BC_GHOST, halo_lo=top, halo_hi=bot,
                  halo_lo_offset=shift * es, halo_hi_offset=shift * es, halo_width=len(halo[0]))
    off = dict(in_offset=shift * es, out_offset=shift * es, tmp_offset=shift * es)
    args = hx.stencil_args(dims=2, dtype=hx.HX_F64 if dt == np.float64 else hx.HX_F32, nx=nx,
                           ny=ny, steps=steps, r=r, inp=bi, out=bo, tmp=bt, **off, **kw, **geom)
    run(ctx, args)
    res = download(ctx, bo, (ny, nx), dt, offset=shift * es)
    for b in bufs:
        hx.hx_buffer_destroy(ctx, b)
    return res


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("r", [0.2, 0.25])
def test_forms_give_the_same_bits(ctx, dtype, shape, r):
    u0 = workloads.uniform(shape, 910, shape[0] * 2000 + shape[1], -1, 1, dtype)
    hx.hx_tune_cache_clear()
    for depth, shift in ((1, 0), (3, 1), (8, 0), (7, 3)):
        steps = 2 * depth + 1
        tile = grid(ctx, u0, r, steps, shift, time_block=depth)
        stream = grid(ctx, u0, r, steps, shift, time_block=depth, rows_per_block=9)
        assert np.array_equal(tile, stream), (depth, shift)
        ref = oracle.heat2d_dirichlet(u0.astype(np.float64), r, steps)
        assert rel_l2(tile, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("steps", [9, 24, 31, 100])
def test_library_depths(ctx, dtype, steps):
    """Depths of the library's choosing (up to 24 steps per pass)."""
    for shape in ((70, 300), (257, 129), (600, 1001)):
        u0 = workloads.uniform(shape, 911, shape[0], 0, 1, dtype)
        got = grid(ctx, u0, 0.2, steps)
        ref = oracle.heat2d_dirichlet(u0.astype(np.float64), 0.2, steps)
        assert rel_l2(got, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("nx", [256, 301])
def test_halo_rows(ctx, dtype, nx):
    """Halo-fed bands: both forms read the same halo rows and nothing past them."""
    full = workloads.uniform((60, nx), 912, nx, 0, 1, dtype)
    band, top, bot = full[20:45], full[12:20], full[45:53]
    for depth in (1, 5, 8):
        a = grid(ctx, band, 0.2, depth, 1, halo=(top, bot))
        b = grid(ctx, band, 0.2, depth, 1, halo=(top, bot), rows_per_block=7)
        assert np.array_equal(a, b)
        ref = oracle.heat2d_dirichlet(full.astype(np.float64), 0.2, depth)[20:45]
        assert rel_l2(a, ref) <= TOL[dtype]


def test_non_finite_cells_stay_in_their_light_cone(ctx):
    u0 = workloads.uniform((80, 520), 913, 0, 0, 1, np.float32)
    u0[40, 250] = np.nan
    u0[10, 400] = np.inf
    got = grid(ctx, u0, 0.2, 6, time_block=6)
    y, x = np.mgrid[:80, :520]
    reach = (abs(y - 40) + abs(x - 250) <= 6) | (abs(y - 10) + abs(x - 400) <= 6)
    assert not np.isfinite(got[reach]).any() and np.isfinite(got[~reach]).all()


def test_a_multi_pass_run_still_needs_tmp(ctx):
    """Nine steps needed tmp before deeper passes existed, and still do."""
    u0 = np.zeros((16, 16), np.float32)
    a, b = upload(ctx, u0), hx.hx_buffer_create(ctx, u0.nbytes)
    kw = dict(dims=2, dtype=hx.HX_F32, nx=16, ny=16, r=0.2, inp=a, out=b,
              bc_lo=hx.HX_BC_DIRICHLET0, bc_hi=hx.HX_BC_DIRICHLET0)
    run(ctx, hx.stencil_args(steps=8, **kw))
    with pytest.raises(hx.HxError):
        hx.hx_launch_stencil(ctx, hx.stencil_args(steps=9, **kw))
