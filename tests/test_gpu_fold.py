"""GPU parity of the folded split-precision grid sum (the hi+lo methods' default evaluation) at
the edges of its blocks: x extents around the 64- and 128-column blocks and their mirror, row
counts around the 128 rows, operand waves whose 64 rows lie in one z-slice or cross several, mode
counts around the 16-mode stages and their padding to 64, launches with and without mode slices."""
import ctypes

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


@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n", [((1, 1), 5), ((2, 130), 64), ((127, 129), 65), ((128, 128), 16), ((129, 127), 200),
                                     ((255, 3), 1), ((257, 70), 300), ((700, 260), 129), ((5, 4, 3), 7),
                                     ((65, 64, 4), 64), ((64, 63, 5), 100), ((130, 128, 3), 257), ((260, 10, 14), 33),
                                     ((20, 1, 200), 48), ((100, 192, 9), 520)])
def test_fold_edges(orc, grf, shape, n, meth):
    print(f"case fold {shape} n={n} {meth}", flush=True)
    dim = len(shape)
    ell, sigma = (6.0, 5.0, 2.0)[:dim], 1.3
    geo = dict(origin=(0.5, -30.0, 2.0)[:dim], h=(1.0, 1.5, 0.75)[:dim])
    z, phi = orc.sample_modes(dim, wl.EXPONENTIAL, n, 4400 + n)
    w = 0.25 + np.abs(wl.upstream_grad(n, 4401 + n))
    m = grf.modes_from_tables(z, phi, sigma, ell, w=w)
    C = int(np.prod(shape))
    out = grf.field_grid(m, shape, method=meth, mu=0.1, thresholds=[0.0], want_k=True, want_ind=True, **geo)
    y = to_np(out["y"])
    assert np.isfinite(y).all()
    cells = np.arange(C) if C <= 20000 else wl.sample_cells(C, 6000, 4402)
    scale = sigma * float(np.sqrt(np.mean(w * w)))  # the weighted field's standard deviation
    ref = orc.field_points_w(z, phi, w, sigma, ell, orc.grid_centres(shape, **geo)[cells])
    assert_field(y[cells], ref, scale, meth, f"{shape}")
    np.testing.assert_array_equal(to_np(out["ind"]), (y > 0.0).astype(np.uint8))
    np.testing.assert_allclose(to_np(out["k"]), np.exp(0.1 + y.astype(np.float64)), rtol=1e-6)


def test_fold_without_room_for_slices(orc, grf):
    """A workspace that holds the tables only runs unsplit: the same field up to the FP32
    summation order."""
    shape, n = (150, 97, 21), 700
    print(f"case fold workspace {shape}", flush=True)
    z, phi = orc.sample_modes(3, wl.EXPONENTIAL, n, 4500)
    m = grf.modes_from_tables(z, phi, 1.0, (9.0, 7.0, 3.0))
    from paper_2212_10961_amd import _lib as L
    C = int(np.prod(shape))
    full = grf.grid_workspace_bytes(m, shape, "sep_f16_x3")
    split = grf.field_grid(m, shape, method="sep_f16_x3")["y"]
    small = torch.empty(full - 4 * C, dtype=torch.uint8, device="cuda")
    ya = torch.empty(C, device="cuda")
    mc, gc, ec = m.c(), grf._grid(shape), grf._epi(None, None)
    assert L.load().eval_field_grid(ctypes.byref(mc), ctypes.byref(gc), L.GRF_SEP_F16_X3, ctypes.byref(ec),
                                    ctypes.c_void_p(ya.data_ptr()), None, None, ctypes.c_void_p(small.data_ptr()),
                                    small.numel(), None) == 0
    a, b = to_np(ya), to_np(split)
    cells = wl.sample_cells(C, 3000, 4501)
    ref = orc.field_cells(z, phi, 1.0, (9.0, 7.0, 3.0), shape, cells)
    for v in (a, b):
        assert_field(v[cells], ref, 1.0, "sep_f16_x3", "unsplit / split")
    assert not np.array_equal(a, b)  # the two really took different routes
