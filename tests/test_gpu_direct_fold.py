"""GPU parity of the direct grid sums' folded contraction at the edges of its tiles: x extents
around the mirrored column tiles, row counts around the row tiles, mode counts around the
eight chunks, the 64-mode stages and the matrix steps, with and without weights."""
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


def _case(orc, grf, shape, n, weighted, seed):
    dim = len(shape)
    ell, sigma = (6.0, 5.0, 2.0)[:dim], 1.3
    geo = dict(origin=(0.5, -300.0, 2.0)[:dim], h=(1.0, 1.5, 0.75)[:dim])
    z, phi = orc.sample_modes(dim, wl.EXPONENTIAL, n, seed)
    w = 0.25 + np.abs(wl.upstream_grad(n, seed + 1)) if weighted else None
    m = grf.modes_from_tables(z, phi, sigma, ell, w=w)
    return z, phi, (np.ones(n) if w is None else w), m, sigma, ell, geo


@pytest.mark.parametrize("meth", ["direct_f32", "direct_f64"])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("shape,n", [((1, 1), 1), ((2, 3), 2), ((3, 1, 1), 7), ((31, 17), 8), ((32, 16), 9),
                                     ((33, 15, 3), 63), ((63, 9, 2), 64), ((64, 4, 4), 65), ((65, 33), 511),
                                     ((300, 41), 513), ((129, 130, 5), 130), ((70, 64, 110), 37)])
def test_direct_grid_edges(orc, grf, shape, n, weighted, meth):
    print(f"case direct fold {shape} n={n} weighted={weighted} {meth}", flush=True)
    z, phi, w, m, sigma, ell, geo = _case(orc, grf, shape, n, weighted, 4100 + n)
    C = int(np.prod(shape))
    out = grf.field_grid(m, shape, method=meth, mu=0.1, thresholds=[0.0], want_k=True, want_ind=True, **geo)
    y = to_np(out["y"])
    cells = np.arange(C) if C <= 20000 else wl.sample_cells(C, 5000, 4200)
    ref = orc.field_points_w(z, phi, w, sigma, ell, orc.grid_centres(shape, **geo)[cells])
    scale = sigma * float(np.sqrt(np.mean(w * w)))  # the weighted field's standard deviation
    assert_field(y[cells], ref, scale, meth, f"{shape}")
    assert np.isfinite(y).all()
    np.testing.assert_array_equal(to_np(out["ind"]), (y > 0.0).astype(np.uint8))
    np.testing.assert_allclose(to_np(out["k"]), np.exp(0.1 + y.astype(np.float64)), rtol=1e-6)


@pytest.mark.parametrize("shape", [(40, 30), (200, 190), (300, 450), (128, 100, 60)])
def test_direct_tiles_agree_with_batch(orc, grf, shape):
    """Every tile the size rule picks gives the batched evaluation's bits (whole grids, 517 modes:
    chunks of 72 modes, the last of 13)."""
    print(f"case direct fold batch {shape}", flush=True)
    z, phi, w, m, sigma, ell, geo = _case(orc, grf, shape, 517, True, 4300)
    y = torch.empty(int(np.prod(shape)), device="cuda")
    plan = grf.Plan("direct_f32", graph=False, autotune=False)
    plan.run([(m, shape, y)])
    np.testing.assert_array_equal(to_np(grf.field_grid(m, shape)["y"]), to_np(y))
    plan.close()
