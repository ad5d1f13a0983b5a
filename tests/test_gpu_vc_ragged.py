"""The fused variable-coefficient passes on grids whose rows are no multiple of
the vector width or start off 16 bytes: the same bits as the run composed of
single steps, and the oracle's gradient."""
import numpy as np
import pytest

import oracle
import workloads
from conftest import rel_l2

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, upload  # noqa: E402

# around the strip's 248 columns and the lane's 4; 3 columns take single steps
SHAPES = [(1, 4), (2, 5), (9, 3), (40, 247), (13, 249), (50, 250), (7, 251), (70, 497), (33, 1003),
          (64, 256)]


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


def fields(shape, dtype):
    ny, nx = shape
    u0 = workloads.uniform(shape, 920, ny * 5000 + nx, 0, 1, dtype)
    kap = workloads.uniform(shape, 921, ny * 5000 + nx, 0.05, 1, dtype)
    lam = workloads.uniform(shape, 922, ny * 5000 + nx, -1, 1, dtype)
    return u0, kap, lam


class Dev:
    """Buffers of one run; every operand starts `shift` cells into its allocation."""

    def __init__(self, ctx, shape, dtype, shift):
        self.ctx, self.shape, self.dtype, self.shift = ctx, shape, dtype, shift
        self.cells, self.es = shape[0] * shape[1], np.dtype(dtype).itemsize
        self.bufs = []

    def new(self, states, arr=None, es=None):
        es = es or self.es
        raw = hx.hx_buffer_create(self.ctx, (states * self.cells + self.shift) * es)
        ptr, _ = hx.hx_buffer_ptr(self.ctx, raw)
        b = hx.hx_buffer_wrap(self.ctx, ptr + self.shift * es, max(states * self.cells * es, es))
        self.bufs += [b, raw]
        if arr is not None:
            e = hx.hx_copy_async(self.ctx, hx.hx_copy_desc(hx.HX_H2D, arr.ctypes.data, b, 0, 0, 0,
                                                           arr.nbytes))
            assert hx.hx_wait(self.ctx, e) == hx.HX_OK
        return b

    def get(self, b, dtype=None):
        return download(self.ctx, b, self.shape, dtype or self.dtype)

    def close(self):
        for b in self.bufs:
            hx.hx_buffer_destroy(self.ctx, b)


def gradient(ctx, shape, dtype, T, S, shift, rows=0):
    u0, kap, lam = fields(shape, dtype)
    d = Dev(ctx, shape, dtype, shift)
    code = hx.HX_F64 if dtype == np.float64 else hx.HX_F32
    seg, nseg = hx.hx_vc_schedule(T, S)
    a = hx.hx_vc_args(code, shape[1], shape[0], 0.2, T, S, d.new(1, u0), d.new(1, kap), d.new(1),
                      d.new(max(nseg - 1, 1)), d.new(2), d.new(max(seg - 1, 1)), d.new(1, lam),
                      d.new(1), d.new(1, es=8), d.new(1), rows)
    e = hx.hx_heat_vc_forward(ctx, a)
    e2 = hx.hx_heat_vc_backward(ctx, a, [e])
    assert hx.hx_wait(ctx, e2) == hx.HX_OK, hx.hx_last_error(ctx)
    res = d.get(a.uT), d.get(a.lam0), d.get(a.gk64, np.float64)
    d.close()
    return res


def stepped(ctx, shape, dtype, T, S):
    """The same run from single forward and adjoint steps, folded per segment."""
    u0, kap, lam = fields(shape, dtype)
    code = hx.HX_F64 if dtype == np.float64 else hx.HX_F32
    ny, nx = shape
    k = upload(ctx, kap)
    st = [upload(ctx, u0)]

    def done(e):
        assert hx.hx_wait(ctx, e) == hx.HX_OK

    for _ in range(T):
        st.append(hx.hx_buffer_create(ctx, u0.nbytes))
        done(hx.hx_heat_vc_step(ctx, code, nx, ny, 0.2, st[-2], k, st[-1]))
    uT = download(ctx, st[-1], shape, dtype)
    lams = [upload(ctx, lam), hx.hx_buffer_create(ctx, lam.nbytes)]
    total = np.zeros(shape)
    for s0 in reversed(range(0, T, S)):
        g = upload(ctx, np.zeros(shape, dtype))
        for t in reversed(range(s0, min(s0 + S, T))):
            done(hx.hx_heat_vc_adjoint_step(ctx, code, nx, ny, 0.2, st[t], lams[0], k, lams[1], g))
            lams.reverse()
        total += download(ctx, g, shape, dtype).astype(np.float64)
        hx.hx_buffer_destroy(ctx, g)
    lam0 = download(ctx, lams[0], shape, dtype)
    for b in st + lams + [k]:
        hx.hx_buffer_destroy(ctx, b)
    return uT, lam0, total


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", SHAPES)
def test_fused_equals_single_steps(ctx, dtype, shape):
    for T, S in ((7, 3), (9, 5), (4, 1)):
        want = stepped(ctx, shape, dtype, T, S)
        for shift, rows in ((0, 0), (1, 0), (0, 5)):
            got = gradient(ctx, shape, dtype, T, S, shift, rows)
            for x, y in zip(got, want):
                assert np.array_equal(x, y), (T, S, shift, rows)


@pytest.mark.parametrize("dtype,tol", [(np.float32, 1e-5), (np.float64, 1e-12)])
@pytest.mark.parametrize("shape", [(61, 129), (200, 1001)])
def test_gradient_matches_oracle(ctx, dtype, tol, shape):
    """dL/du0 and dL/dkappa of L = 0.5 ||u_T - y||^2 against the oracle."""
    u0, kap, _ = fields(shape, dtype)
    y = workloads.uniform(shape, 923, shape[0], 0, 1, dtype)
    T = 12
    f64 = [v.astype(np.float64) for v in (u0, kap, y)]
    ref = oracle.heatvc_grad(*f64, 0.2, T, 4)
    import torch
    from paper_1810_11482_amd.adjoint import HeatLoss, HeatVC
    tu, tk, ty = (torch.from_numpy(v).cuda() for v in (u0, kap, y))
    tu.requires_grad_()
    tk.requires_grad_()
    with torch.cuda.stream(torch.cuda.Stream()):
        torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
        loss = HeatLoss.apply(HeatVC.apply(tu, tk, 0.2, T, 4), ty)
        gu, gk = torch.autograd.grad(loss, (tu, tk))
        torch.cuda.synchronize()
    assert abs(float(loss.detach()) - ref[0]) <= tol * abs(ref[0])
    assert rel_l2(gu.cpu().numpy(), ref[1]) <= tol
    assert rel_l2(gk.cpu().numpy(), ref[2]) <= tol
