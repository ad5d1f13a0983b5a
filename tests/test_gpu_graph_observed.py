"""A partitioned f32 graph gives the same bits whether its nodes are watched or
not: without node events (whole passes), with them, under the hazard checker
and captured into a graph; at sizes and depths where a pass takes the propagator
form as well as where it is stepped, and in groups of partitions that differ."""
import numpy as np
import pytest

import oracle
import workloads
from conftest import rel_l2

pytestmark = pytest.mark.gpu
hx = pytest.importorskip("paper_1810_11482_amd")
from hxutil import download, upload  # noqa: E402

CASES = [  # sizes, steps, time_block, rate
    ([300000] * 16, 50, 0, 0.25),
    ([40000 + 13 * k for k in range(70)], 150, 100, 0.25),
    ([4096, 5000, 70001, 256 + 4096], 64, 32, 0.2),
    ([256] * 5 + [300000] * 4, 200, 200, 0.1),
    ([2000000, 1000001], 41, 20, 0.05),
    ([1000] * 65 + [1 << 21], 128, 64, 0.25),
    ([1 << 20], 70, 33, 0.25),
]


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_same_bits(case, periodic):
    if hx.hx_device_count() == 0:
        pytest.skip("no GPU")
    hx.hx_tune_cache_clear()
    sizes, steps, tb, r = CASES[case]
    if len(sizes) == 1 and not periodic:
        pytest.skip("an ordinary run")
    n, off = sum(sizes), np.cumsum([0] + sizes)
    u0 = workloads.uniform(n, 980, case, 0, 1, np.float32)
    runs = {}
    for how in ("whole", "nodes", "checked", "captured"):
        ctx = hx.hx_ctx_create(0, check=how == "checked")
        raw = [upload(ctx, np.concatenate([np.zeros(3, np.float32), u0])),
               hx.hx_buffer_create(ctx, u0.nbytes + 12)]
        sets = [[hx.hx_buffer_wrap(ctx, hx.hx_buffer_ptr(ctx, b)[0] + 12 + 4 * int(o), 4 * m)
                 for o, m in zip(off, sizes)] for b in raw]
        d = hx.partitioned_desc(hx.HX_F32, sizes, *sets, steps, r, periodic=periodic, time_block=tb)
        if how == "captured":
            hx.hx_graph_begin(ctx)
        ev, in_b, _ = hx.hx_run_partitioned(ctx, d, node_events=how == "nodes")
        if how == "captured":
            hx.hx_event_release(ctx, ev)
            graph = hx.hx_graph_end(ctx)
            ev = hx.hx_graph_launch(ctx, graph)
        assert hx.hx_wait(ctx, ev) == hx.HX_OK, hx.hx_last_error(ctx)
        runs[how] = download(ctx, raw[int(in_b)], n, np.float32, offset=12)
        if how == "checked":
            assert hx.hx_hazard_count(ctx) == 0
        hx.hx_ctx_destroy(ctx)
    for how in ("nodes", "checked", "captured"):
        assert np.array_equal(runs["whole"], runs[how]), how
    f = oracle.heat1d_periodic if periodic else oracle.heat1d_dirichlet
    assert rel_l2(runs["whole"], f(u0.astype(np.float64), r, steps)) <= 1e-5
