"""Grids one cell wide along x (and y): the direct and hi+lo sums fold the first axis with more cells,
on grids and in batches, with weights, rotations, spacings and all outputs."""
import numpy as np
import pytest
import torch

from gpu_common import assert_field, to_np
from paper_2212_10961_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_10961_amd.grf as g
    return g


SHAPES = [(1, 1), (1, 50), (1, 3000), (1, 1, 1), (1, 1, 77), (1, 37, 21), (1, 300, 5), (1, 2, 400), (3, 1, 40)]


@pytest.mark.parametrize("meth", ["direct_f32", "direct_f64", "sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_cell_axes(orc, grf, shape, meth):
    print(f"case one-cell axes {shape} {meth}", flush=True)
    dim, n = len(shape), 230
    ell, sigma = (6.0, 5.0, 2.0)[:dim], 1.3
    geo = dict(origin=(0.5, -300.0, 2.0)[:dim], h=(1.0, 1.5, 0.75)[:dim])
    z, phi = orc.sample_modes(dim, wl.EXPONENTIAL, n, 5700)
    w = 0.25 + np.abs(wl.upstream_grad(n, 5701))
    m = grf.modes_from_tables(z, phi, sigma, ell, w=w)
    out = grf.field_grid(m, shape, method=meth, mu=0.1, thresholds=[0.0], want_k=True, want_ind=True, **geo)
    y = to_np(out["y"])
    scale = sigma * float(np.sqrt(np.mean(w * w)))
    x = orc.grid_centres(shape, **geo)
    assert_field(y, orc.field_points_w(z, phi, w, sigma, ell, x), scale, meth, f"{shape}")
    np.testing.assert_array_equal(to_np(out["ind"]), (y > 0.0).astype(np.uint8))
    np.testing.assert_allclose(to_np(out["k"]), np.exp(0.1 + y.astype(np.float64)), rtol=1e-6)
    a = 0.7
    rot = np.eye(3)
    rot[:2, :2] = [[np.cos(a), -np.sin(a)], [np.sin(a), np.cos(a)]]
    mr = grf.modes_from_tables(z, phi, sigma, ell, rot=rot[:dim, :dim])
    yr = to_np(grf.field_grid(mr, shape, method=meth, **geo)["y"])
    assert_field(yr, orc.field_points_mat(z, phi, sigma, rot[:dim, :dim] / np.array(ell), x), sigma, meth, f"{shape} rotated")
    if meth == "direct_f32":  # a batch of the same grids: the same bits
        yb = torch.empty(y.size, device="cuda")
        plan = grf.Plan("direct_f32", graph=False, autotune=False)
        plan.run([(m, shape, yb)])
        np.testing.assert_array_equal(to_np(grf.field_grid(m, shape, method=meth)["y"]), to_np(yb))
        plan.close()
    if meth == "direct_f64":
        y64 = to_np(grf.field_grid_f64(m, shape, mu=0.0, **geo)["y"])
        assert np.max(np.abs(y64 - orc.field_points_w(z, phi, w, sigma, ell, x))) <= 1e-11 * scale


@pytest.mark.parametrize("rows", [1, 16, 20, 32, 33])
def test_f64_few_rows(orc, grf, rows):
    """FP64 sums over few long rows: one or four row tiles per block."""
    print(f"case few rows {rows}", flush=True)
    shape, ell = (8200, rows), (6.0, 5.0)
    z, phi = orc.sample_modes(2, wl.EXPONENTIAL, 70, 5720)
    m = grf.modes_from_tables(z, phi, 1.3, ell)
    y64 = to_np(grf.field_grid_f64(m, shape)["y"])
    assert np.max(np.abs(y64 - orc.field_grid(z, phi, 1.3, ell, shape))) <= 1e-11 * 1.3


@pytest.mark.parametrize("n", [64, 1000])
def test_f64_time_does_not_depend_on_the_axis(grf, n):
    """FP64 sums over the same 65,536 cells along (y, z) and along (x, y): at most 1.3 times the time
    (graphs of ten calls, best of seven)."""
    print(f"case one-cell axes time n={n}", flush=True)
    m = grf.modes_from_tables(*grf.make_modes(3, wl.GAUSSIAN, n, 5710), 1.0, (9.0, 9.0, 9.0))

    def graph(shape):
        grf.field_grid_f64(m, shape)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(10):
                grf.field_grid_f64(m, shape)
        return g

    def once(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b) / 10 * 1e3

    gs = [graph((1, 256, 256)), graph((256, 256, 1))]
    t = np.array([[once(g) for g in gs] for _ in range(8)])[1:].min(axis=0)
    print(f"  1 x 256 x 256 {t[0]:.1f} us, 256 x 256 x 1 {t[1]:.1f} us", flush=True)
    assert t[0] <= 1.3 * t[1]
