"""The FP32 grid sum's three tiles (64 rows x 32 columns, 32 x 32, 16 x 16; a column is a cell and its
mirror): grids that the size rule gives to each, with and without weights, agree bit for bit with
the batch's 64 x 32 tile and with the oracle.

Tolerance: a phase is formed and reduced in FP64 and rounded once (2^-25 revolutions, 2e-7 in a
cosine), the hardware cosine and sine add 1.2e-7 each, an FP32 product and FMA per term round at
2^-24 of partial sums of a chunk's modes: a few 1e-7 of sigma in all, far inside the bar of the
direct form (relative 2e-5, 1e-4 sigma)."""
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


def _tile(shape):
    """The size rule: at least 160 tiles of 64 x 32, else at least 192 of 32 x 32, else 16 x 16."""
    half, rows = (shape[0] + 1) // 2, int(np.prod(shape[1:]))

    def tiles(r, c):
        return -(-half // c) * -(-rows // r)

    return 64 if tiles(64, 32) >= 160 else (32 if tiles(32, 32) >= 192 else 16)


CASES = {(150, 97, 21): 32, (300, 270, 5): 32, (1024, 512): 32, (64, 98, 64): 32, (512, 512, 4): 64, (300, 270, 9): 64,
         (1025, 640): 64, (70, 45, 9): 16, (517, 301): 16, (64, 64, 64): 16}


def test_cases_span_the_rule():
    assert {s: _tile(s) for s in CASES} == CASES and set(CASES.values()) == {16, 32, 64}


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("shape", list(CASES))
def test_tiles_match_batch(orc, grf, shape, weighted):
    print(f"case direct tiles {shape} weighted={weighted}", flush=True)
    dim, n = len(shape), 331
    ell = (7.0, 5.0, 2.0)[:dim]
    z, phi = orc.sample_modes(dim, wl.EXPONENTIAL, n, 5800)
    w = 0.25 + np.abs(wl.upstream_grad(n, 5801)) if weighted else None
    m = grf.modes_from_tables(z, phi, 1.1, ell, w=w)
    C = int(np.prod(shape))
    yb = torch.empty(C, device="cuda")
    plan = grf.Plan("direct_f32", graph=False, autotune=False)
    plan.run([(m, shape, yb)])
    y = to_np(grf.field_grid(m, shape, method="direct_f32")["y"])
    np.testing.assert_array_equal(y, to_np(yb), err_msg=f"{shape}")
    plan.close()
    cells = wl.sample_cells(C, 3000, 5802)
    w = np.ones(n) if w is None else w
    ref = orc.field_points_w(z, phi, w, 1.1, ell, orc.grid_centres(shape)[cells])
    assert_field(y[cells], ref, 1.1 * float(np.sqrt(np.mean(w * w))), "direct_f32", f"{shape}")
