"""GPU parity of the separable adjoint where its kernel takes one and two mode groups per wave, at
the edges of its tiles: row chunks left without a tile, slices of several 32-row
tiles with padded rows, a second x chunk, mode counts that leave padding in the last group."""
import numpy as np
import pytest
import torch

from gpu_common import modes_pair, to_np
from paper_2212_10961_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_10961_amd.grf as g
    return g


def _rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


# one group, then (four tiles and more per row chunk) two
@pytest.mark.parametrize("shape,n", [((33, 31, 7), 129), ((9, 70, 90), 64), ((130, 33, 130), 100),
                                     ((130, 5, 1030), 100), ((17, 33, 515), 65), ((3, 33000), 128), ((5, 70, 60), 1100)])
def test_mode_groups(orc, grf, shape, n):
    dim = len(shape)
    ell, sigma = (9.0, 4.0, 2.0)[:dim], 0.9
    print(f"case adjoint groups {shape} n={n}", flush=True)
    (zo, po), m = modes_pair(orc, grf, dim, wl.GAUSSIAN, n, 1140 + n, sigma, ell)
    C = int(np.prod(shape))
    g = wl.upstream_grad(C, 1141).astype(np.float32)
    geo = dict(origin=(0.5, -3.0, 2.0)[:dim], h=(1.0, 0.7, 1.5)[:dim])
    ref = orc.grad_points(zo, po, sigma, ell, orc.grid_centres(shape, **geo), g.astype(np.float64))
    out = grf.field_backward_grid(m, shape, torch.from_numpy(g).cuda(), method="sep_bf16_x3", **geo)
    # per mode: the dropped lo x lo product and the operands' own rounding, 2^-16 each and more
    # terms than that spread; the two scalars are sums over modes that cancel
    assert _rel(to_np(out["dphi"]), ref["dphi"]) <= 5e-5
    assert _rel(to_np(out["dk"]), ref["dk"]) <= 5e-5
    assert _rel(to_np(out["dsigma"]), [ref["dsigma"]]) <= 5e-4
    assert _rel(to_np(out["dell"]), ref["dell"]) <= 5e-4
