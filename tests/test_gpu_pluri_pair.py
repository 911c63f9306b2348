"""Bitruncated facies by the hi+lo methods: both fields' tables and sums by one launch each, with and
without mode slices; pairs of tables of different lengths; the time beside two separate fields."""
import numpy as np
import pytest
import torch

from gpu_common import assert_field, modes_pair, to_np
from paper_2212_10961_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_10961_amd.grf as g
    return g


def _rule(grf):
    return grf.trunc2([-1.0, 0.0, 1.0], [-0.5, 0.5], np.arange(12, dtype=np.uint8).reshape(4, 3) % 5,
                      np.arange(5, dtype=np.float32) + 0.5)


@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n1,n2", [((1, 1), 300, 300), ((257, 129), 517, 550), ((700, 260), 64, 33),
                                         ((31, 9, 5), 1000, 1000), ((130, 128, 3), 100, 100), ((40, 30, 60), 700, 300),
                                         ((256, 256, 40), 70, 128), ((300, 200), 64, 700)])
def test_pair(orc, grf, shape, n1, n2, meth):
    dim = len(shape)
    print(f"case pluri pair {shape} n={n1},{n2} {meth}", flush=True)
    l1, l2 = (9.0, 5.0, 2.0)[:dim], (6.0, 6.0, 3.0)[:dim]
    (z1, p1), m1 = modes_pair(orc, grf, dim, wl.GAUSSIAN, n1, 5400 + n1, 1.4, l1)
    (z2, p2), m2 = modes_pair(orc, grf, dim, wl.EXPONENTIAL, n2, 5500 + n2, 1.0, l2)
    rule = _rule(grf)
    kept = grf.pluri_grid(m1, m2, shape, rule, method=meth, want_value=True, keep_fields=True)
    C = int(np.prod(shape))
    cells = np.arange(C) if C <= 20000 else wl.sample_cells(C, 4000, 5401)
    assert_field(to_np(kept["y1"])[cells], orc.field_cells(z1, p1, 1.4, l1, shape, cells), 1.4, meth, f"{shape} y1")
    assert_field(to_np(kept["y2"])[cells], orc.field_cells(z2, p2, 1.0, l2, shape, cells), 1.0, meth, f"{shape} y2")
    want = grf.pluri_apply(kept["y1"], kept["y2"], rule, want_value=True)
    lost = grf.pluri_grid(m1, m2, shape, rule, method=meth, want_value=True)
    for out in (kept, lost):
        np.testing.assert_array_equal(to_np(out["facies"]), to_np(want["facies"]))
        np.testing.assert_array_equal(to_np(out["value"]), to_np(want["value"]))


@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n", [((256, 128), 64), ((1024, 512), 64), ((512, 256), 1000)])
def test_pair_is_no_slower_than_two_fields(grf, shape, n, meth):
    """At most the time of both fields by explicit separable tiles and the rule (graphs of 20 calls,
    best of seven)."""
    print(f"case pluri pair time {shape} n={n} {meth}", flush=True)
    m1 = grf.modes_from_tables(*grf.make_modes(2, wl.GAUSSIAN, n, 5600), 1.0, (9.0, 7.0))
    m2 = grf.modes_from_tables(*grf.make_modes(2, wl.EXPONENTIAL, n, 5601), 1.0, (9.0, 7.0))
    rule = _rule(grf)
    C = int(np.prod(shape))
    ws = torch.empty(grf.grid_workspace_bytes(m1, shape, meth), dtype=torch.uint8, device="cuda")
    y1, y2 = torch.empty(C, device="cuda"), torch.empty(C, device="cuda")

    def pair():
        grf.pluri_grid(m1, m2, shape, rule, method=meth, want_value=True)

    def two(tile):
        def run():
            for m, y in ((m1, y1), (m2, y2)):
                grf.field_grid(m, shape, method=meth, tile=tile, out={"y": y}, workspace=ws)
            grf.pluri_apply(y1, y2, rule, want_value=True)
        return run

    def graph(run):
        run()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                run()
        return g

    def once(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b) / 20 * 1e3

    gs = [graph(r) for r in (pair, two(2), two(1))]
    t = np.array([[once(g) for g in gs] for _ in range(8)])[1:].min(axis=0)
    print(f"  pair {t[0]:.1f} us, two fields {t[1]:.1f} and {t[2]:.1f} us", flush=True)
    assert t[0] <= min(t[1], t[2])
