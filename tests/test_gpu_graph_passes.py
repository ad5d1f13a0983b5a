"""A partitioned graph whose nodes the caller does not ask for takes each pass
in launches of many partitions: the same bits as the graph of one node per
partition and pass, for any sizes, boundaries, depths and numbers of parts."""
import numpy as np
import pytest

import oracle
import workloads
from conftest import rel_l2

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, upload  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    hx.hx_tune_cache_clear()
    c = hx.hx_ctx_create(0)
    yield c
    hx.hx_ctx_destroy(c)


def graph(ctx, u0, sizes, steps, r, nodes, shift=0, **kw):
    """One run over partitions of `sizes` units, carved out of one allocation
    (so they start at any alignment)."""
    unit = u0.size // sum(sizes)
    es = u0.itemsize
    raw = [upload(ctx, np.concatenate([np.zeros(shift, u0.dtype), u0.ravel()])),
           hx.hx_buffer_create(ctx, u0.nbytes + shift * es)]
    sets = []
    for b in raw:
        ptr, off, bufs = hx.hx_buffer_ptr(ctx, b)[0] + shift * es, 0, []
        for m in sizes:
            bufs.append(hx.hx_buffer_wrap(ctx, ptr + off * unit * es, m * unit * es))
            off += m
        sets.append(bufs)
    d = hx.partitioned_desc(hx.HX_F64 if u0.dtype == np.float64 else hx.HX_F32, sizes, *sets,
                            steps, r, **kw)
    ev, in_b, evs = hx.hx_run_partitioned(ctx, d, node_events=nodes)
    assert hx.hx_wait(ctx, ev) == hx.HX_OK, hx.hx_last_error(ctx)
    for e in [ev] + (evs or []):
        hx.hx_event_release(ctx, e)
    res = download(ctx, raw[int(in_b)], u0.shape, u0.dtype.type, offset=shift * es)
    for b in sets[0] + sets[1] + raw:
        hx.hx_buffer_destroy(ctx, b)
    return res


@pytest.mark.parametrize("dtype,tol", [(np.float32, 1e-5), (np.float64, 1e-12)])
@pytest.mark.parametrize("periodic", [True, False])
def test_1d_passes_equal_nodes(ctx, dtype, tol, periodic):
    g = np.random.default_rng(5)
    for parts, lo, hi in ((1, 200, 200), (2, 64, 70), (16, 64, 3000), (65, 64, 400),
                          (130, 64, 90)):
        sizes = [int(x) for x in g.integers(lo, hi + 1, parts)]
        u0 = workloads.uniform(sum(sizes), 940, parts, 0, 1, dtype)
        f = oracle.heat1d_periodic if periodic else oracle.heat1d_dirichlet
        for steps, tb, r in ((50, 0, 0.25), (64, 64, 0.2), (7, 3, 0.45)):
            if (tb or 32) > min(sizes) or (parts == 1 and not periodic and tb > 50):
                continue  # refused: a pass deeper than a partition, or a lone run without tmp
            kw = dict(periodic=periodic, time_block=tb)
            a = graph(ctx, u0, sizes, steps, r, False, shift=parts % 4, **kw)
            b = graph(ctx, u0, sizes, steps, r, True, shift=parts % 4, **kw)
            assert np.array_equal(a, b), (parts, steps, tb)
            assert rel_l2(a, f(u0.astype(np.float64), r, steps)) <= tol


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_2d_passes_equal_nodes(ctx, dtype):
    for sizes, nx in (([20, 33, 9], 300), ([8] * 20, 129)):
        u0 = workloads.uniform((sum(sizes), nx), 941, nx, 0, 1, dtype)
        kw = dict(periodic=False, dims=2, nx=nx)
        a = graph(ctx, u0, sizes, 21, 0.2, False, **kw)
        b = graph(ctx, u0, sizes, 21, 0.2, True, **kw)
        assert np.array_equal(a, b)


def test_errors_are_the_nodes(ctx):
    """What the node form refuses, the whole passes refuse."""
    n = 4096
    a, b = (hx.hx_buffer_create(ctx, n * 4) for _ in range(2))
    for kw in (dict(time_block=5000), dict(cells_per_lane=12), dict(waves_per_group=3),
               dict(cells_per_lane=8, time_block=300)):
        for nodes in (False, True):
            with pytest.raises(hx.HxError):
                hx.hx_run_partitioned(ctx, hx.partitioned_desc(hx.HX_F32, [n], [a], [b], 4000,
                                                               0.2, **kw), node_events=nodes)
    for nodes in (False, True):
        with pytest.raises(hx.HxError):
            hx.hx_run_partitioned(ctx, hx.partitioned_desc(hx.HX_F32, [n], [a], [a], 10, 0.2),
                                  node_events=nodes)


def test_a_failed_dependency_fails_the_graph(ctx):
    n = 4096
    a, b = (hx.hx_buffer_create(ctx, n * 4) for _ in range(2))
    gate = hx.hx_user_event_create(ctx)
    ev, _, _ = hx.hx_run_partitioned(ctx, hx.partitioned_desc(hx.HX_F32, [n // 2] * 2, [a, a],
                                                              [b, b], 40, 0.2), deps=[gate])
    hx.hx_user_event_set(ctx, gate, hx.HX_ERR_ARG)
    assert hx.hx_wait(ctx, ev) == hx.HX_ERR_DEP_FAILED
