"""The fp16 hi+lo form's operands are split from FP64 cosines and sines.

A single mode on one row is the product of two operands (the column's and the row's), each held as an
fp16 pair, with no sum to hide their rounding: the pair's lo word has 11 bits below a remainder of at
most 2^-12 of values up to 1, an error of at most 2^-24 where the remainder is exact; the three
products that are kept leave out lo x lo (2^-24), and FP32 rounds each of four accumulations of values
up to 1 (2^-25) and the final difference.  Rounding the cosine to FP32 first would add 2^-25 per operand.
Root mean square over cells: about 0.3 to 0.5 of each, in all below 5e-8 of the mode's amplitude."""
import numpy as np
import pytest
import torch

from gpu_common import to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_10961_amd.grf as g
    return g


@pytest.mark.parametrize("shape", [(600, 40), (257, 90)])
def test_single_modes(grf, shape):
    print(f"case fold precision {shape}", flush=True)
    rng = np.random.default_rng(5900)
    sq = []
    for _ in range(24):
        z, phi = rng.standard_normal((2, 1)), rng.random(1) * 2 * np.pi
        m = grf.modes_from_tables(z, phi, float(np.sqrt(0.5)), (8.0, 7.0))  # amplitude 1
        y = to_np(grf.field_grid(m, shape, method="sep_f16_x3")["y"]).astype(np.float64)
        ref = to_np(grf.field_grid_f64(m, shape)["y"])
        sq.append(np.mean((y - ref) ** 2))
    rms = float(np.sqrt(np.mean(sq)))
    print(f"  rms {rms:.3e}", flush=True)
    assert rms <= 5e-8
