"""GPU parity of tables of more than 2^19 modes: launches whose mode axis is longer than a grid's
second dimension (65,535 blocks) counts."""
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


# 2^19 modes are the half-space lattice of 1024 points per axis in 2-D, 102^3 / 2 that of 102 in 3-D
@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3", "sep_f16", "direct_f32"])
@pytest.mark.parametrize("shape,n", [((21, 12), 1024 * 512), ((9, 6, 4), 102 * 102 * 51)])
def test_grid_of_many_modes(orc, grf, shape, n, meth):
    print(f"case many modes {shape} n={n} {meth}", flush=True)
    dim = len(shape)
    ell = (6.0, 5.0, 2.0)[:dim]
    z, phi = orc.sample_modes(dim, wl.GAUSSIAN, n, 4600)
    m = grf.modes_from_tables(z, phi, 1.1, ell)
    y = to_np(grf.field_grid(m, shape, method=meth)["y"])
    assert_field(y, orc.field_grid(z, phi, 1.1, ell, shape), 1.1, meth, f"{shape}")
