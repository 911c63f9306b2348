"""The bitruncated rule made straight from both fields' mode-slice sums, around the sizes of a block
and of the slice groups: facies, values and kept fields are those of the separate evaluations."""
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


@pytest.mark.parametrize("shape,n", [((1, 1), 300), ((17, 15), 64), ((64, 4), 2000), ((257, 129), 517), ((31, 9, 5), 4096)])
@pytest.mark.parametrize("keep", [False, True])
def test_rule_from_slice_sums(orc, grf, shape, n, keep):
    dim = len(shape)
    print(f"case pluri slices {shape} n={n} keep={keep}", flush=True)
    _, m1 = modes_pair(orc, grf, dim, wl.GAUSSIAN, n, 5200 + n, 1.4, (9.0, 5.0, 2.0)[:dim])
    _, m2 = modes_pair(orc, grf, dim, wl.EXPONENTIAL, n, 5300 + n, 1.0, (6.0, 6.0, 3.0)[:dim])
    rule = grf.trunc2([-1.0, 0.0, 1.0], [-0.5, 0.5], np.arange(12, dtype=np.uint8).reshape(4, 3) % 5,
                      np.arange(5, dtype=np.float32) + 0.5)
    out = grf.pluri_grid(m1, m2, shape, rule, method="sep_f16", want_value=True, keep_fields=keep)
    y1 = grf.field_grid(m1, shape, method="sep_f16", want_y=True, want_k=False)["y"]
    y2 = grf.field_grid(m2, shape, method="sep_f16", want_y=True, want_k=False)["y"]
    want = grf.pluri_apply(y1, y2, rule, want_value=True)
    np.testing.assert_array_equal(to_np(out["facies"]), to_np(want["facies"]))
    np.testing.assert_array_equal(to_np(out["value"]), to_np(want["value"]))
    if keep:
        np.testing.assert_array_equal(to_np(out["y1"]), to_np(y1))
        np.testing.assert_array_equal(to_np(out["y2"]), to_np(y2))
