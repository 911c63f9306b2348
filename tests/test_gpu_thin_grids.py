"""GPU parity on thin grids with more tiles than a launch's first dimension takes (2^23 blocks
of 512 threads): first and last cells, the cells around the tile counts and random ones."""
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


# 64 cells of a column per block of the FP32 sum, 128 of the hi+lo form
@pytest.mark.parametrize("meth,shape", [("direct_f32", (1, 1 << 24, 33)), ("sep_f16_x3", (1, 1 << 24, 65)),
                                        ("direct_f32", (2, (1 << 24) - 3, 33))])
def test_thin_grid(orc, grf, meth, shape):
    print(f"case thin grid {shape} {meth}", flush=True)
    ell = (3.0, 4000.0, 9.0)
    z, phi = orc.sample_modes(3, wl.GAUSSIAN, 16, 4700)
    m = grf.modes_from_tables(z, phi, 1.0, ell)
    C = int(np.prod(shape))
    y = torch.full((C,), float("nan"), device="cuda")
    grf.field_grid(m, shape, method=meth, out={"y": y})
    assert not bool(torch.isnan(y).any().item())
    rng = np.random.default_rng(4701)
    edges = [64 << 22, 64 << 23, 128 << 22, 128 << 23]
    cells = np.unique(np.concatenate([np.arange(256), np.arange(C - 256, C), rng.integers(0, C, 4096)]
                                     + [np.arange(e - 128, min(e + 128, C)) for e in edges if e < C]))
    ref = orc.field_cells(z, phi, 1.0, ell, shape, cells)
    assert_field(to_np(y[torch.from_numpy(cells).cuda()]), ref, 1.0, meth, f"{shape}")
    del y
    torch.cuda.empty_cache()
