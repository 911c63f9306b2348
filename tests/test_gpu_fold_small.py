"""The hi+lo methods' default evaluation on grids of little work: the stores of a call that asks for Y
alone, tables whose threads take several points, and the time of such calls beside the separable
form's explicit tiles."""
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


def _table(orc, grf, dim, n, seed):
    z, phi = orc.sample_modes(dim, wl.EXPONENTIAL, n, seed)
    w = 0.25 + np.abs(wl.upstream_grad(n, seed + 1))
    ell = (6.0, 5.0, 2.0)[:dim]
    return z, phi, w, ell, grf.modes_from_tables(z, phi, 1.3, ell, w=w)


@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n", [((1, 1), 5), ((2, 130), 64), ((127, 129), 65), ((128, 128), 16), ((255, 3), 1),
                                     ((257, 70), 300), ((700, 260), 129), ((5, 4, 3), 7), ((65, 64, 4), 64),
                                     ((130, 128, 3), 257), ((260, 10, 14), 33), ((20, 1, 200), 48)])
def test_y_alone(orc, grf, shape, n, meth):
    """Y alone, K alone and all three outputs are stored by different loops: the same Y bits, every
    cell written, none outside the buffers."""
    print(f"case fold stores {shape} n={n} {meth}", flush=True)
    z, phi, w, ell, m = _table(orc, grf, len(shape), n, 4800 + n)
    C = int(np.prod(shape))

    def padded(v, dt):
        return torch.full((C + 512,), v, dtype=dt, device="cuda")

    y, k, y3, k3, i3 = (padded(-7.0, torch.float32), padded(-7.0, torch.float32), padded(-7.0, torch.float32),
                        padded(-7.0, torch.float32), padded(77, torch.uint8))
    kw = dict(method=meth, mu=0.1)
    grf.field_grid(m, shape, out={"y": y[256:256 + C]}, **kw)
    grf.field_grid(m, shape, want_y=False, want_k=True, out={"k": k[256:256 + C]}, **kw)
    grf.field_grid(m, shape, want_k=True, want_ind=True, thresholds=[0.0],
                   out={"y": y3[256:256 + C], "k": k3[256:256 + C], "ind": i3[256:256 + C]}, **kw)
    for t, v in ((y, -7.0), (k, -7.0), (y3, -7.0), (k3, -7.0), (i3, 77)):
        t = to_np(t)
        assert (t[:256] == v).all() and (t[256 + C:] == v).all()
    y, y3, k, k3 = (to_np(t)[256:256 + C] for t in (y, y3, k, k3))
    np.testing.assert_array_equal(y, y3)
    np.testing.assert_allclose(k, k3, rtol=1e-6)  # (two exponentials of a few ulp in the separable form)
    cells = np.arange(C) if C <= 20000 else wl.sample_cells(C, 6000, 4801)
    ref = orc.field_points_w(z, phi, w, 1.3, ell, orc.grid_centres(shape)[cells])
    assert_field(y[cells], ref, 1.3 * float(np.sqrt(np.mean(w * w))), meth, f"{shape}")


@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n", [((3001, 40), 520), ((40, 3001), 8000), ((10, 1001, 30), 1100), ((6, 30, 5000), 333)])
def test_tables_of_several_points_per_thread(orc, grf, shape, n, meth):
    print(f"case fold tables {shape} n={n} {meth}", flush=True)
    z, phi, w, ell, m = _table(orc, grf, len(shape), n, 4900 + n)
    C = int(np.prod(shape))
    y = to_np(grf.field_grid(m, shape, method=meth)["y"])
    assert np.isfinite(y).all()
    cells = wl.sample_cells(C, 4000, 4901)
    ref = orc.field_points_w(z, phi, w, 1.3, ell, orc.grid_centres(shape)[cells])
    assert_field(y[cells], ref, 1.3 * float(np.sqrt(np.mean(w * w))), meth, f"{shape}")


@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n", [((256, 256), 64), ((1000, 500), 64), ((2048, 2048), 256), ((256, 256, 64), 256)])
def test_no_slower_than_the_separable_form(grf, shape, n, meth):
    """Calls of few modes: the default evaluation takes at most 1.2 times the better one of the
    separable form's explicit 64 x 64 and 128 x 128 tiles (graphs of 20 calls, best of seven)."""
    print(f"case fold few modes {shape} n={n} {meth}", flush=True)
    dim = len(shape)
    m = grf.modes_from_tables(*grf.make_modes(dim, wl.GAUSSIAN, n, 5000), 1.0, (9.0, 7.0, 3.0)[:dim])
    C = int(np.prod(shape))
    ws = torch.empty(grf.grid_workspace_bytes(m, shape, meth), dtype=torch.uint8, device="cuda")
    y = torch.empty(C, device="cuda")

    def graph(tile):
        kw = dict(method=meth, out={"y": y}, workspace=ws, **({} if tile is None else {"tile": tile}))
        grf.field_grid(m, shape, **kw)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                grf.field_grid(m, shape, **kw)
        return g

    def once(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b) / 20 * 1e3

    gs = [graph(t) for t in (None, 2, 1)]
    t = np.array([[once(g) for g in gs] for _ in range(8)])[1:].min(axis=0)
    print(f"  default {t[0]:.1f} us, tiles {t[1]:.1f} and {t[2]:.1f} us", flush=True)
    assert t[0] <= 1.2 * min(t[1], t[2])
