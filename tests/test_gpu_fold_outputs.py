"""The hi+lo methods' default evaluation with every set of outputs, each stored by a loop of its own:
the same Y bits whatever else is stored, K and facies as they follow from that Y."""
import itertools

import numpy as np
import pytest
import torch

from gpu_common import to_np
from paper_2212_10961_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_10961_amd.grf as g
    return g


@pytest.mark.parametrize("meth", ["sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n", [((1, 1), 3), ((129, 127), 40), ((257, 33, 5), 70), ((96, 96, 96), 100),
                                     ((140, 130, 9), 600)])
def test_output_sets(orc, grf, shape, n, meth):
    print(f"case fold outputs {shape} n={n} {meth}", flush=True)
    z, phi = orc.sample_modes(len(shape), wl.EXPONENTIAL, n, 5100 + n)
    m = grf.modes_from_tables(z, phi, 1.4, (7.0, 6.0, 3.0)[:len(shape)])
    C, mu, thr = int(np.prod(shape)), -0.35, [-1.0, 0.2, 0.9]

    def run(names):
        out = {}
        for name in names:
            dt = torch.uint8 if name == "ind" else torch.float32
            out[name] = torch.full((C + 512,), 91, dtype=dt, device="cuda")
        grf.field_grid(m, shape, method=meth, mu=mu, thresholds=thr, want_y="y" in names, want_k="k" in names,
                       want_ind="ind" in names, out={k: t[256:256 + C] for k, t in out.items()})
        out = {k: to_np(t) for k, t in out.items()}
        for t in out.values():
            assert (t[:256] == 91).all() and (t[256 + C:] == 91).all()
        return {k: t[256:256 + C] for k, t in out.items()}

    y = run(["y"])["y"]
    # expf within one ulp of 2^-23 at most, one more for the rounding of the value compared with
    k = np.exp((np.float32(mu) + y).astype(np.float64))
    ind = (y[:, None] > np.float32(thr)).sum(1)
    for r in (1, 2, 3):
        for names in itertools.combinations(["y", "k", "ind"], r):
            got = run(names)
            if "y" in got:
                np.testing.assert_array_equal(got["y"], y)
            if "k" in got:
                np.testing.assert_allclose(got["k"], k, rtol=2.4e-7)
            if "ind" in got:
                np.testing.assert_array_equal(got["ind"], ind)
