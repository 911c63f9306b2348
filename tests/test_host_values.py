"""The scalars of the differentiable point field as Python floats, whatever types they come in."""
import pytest
import torch

from paper_2212_10961_amd.grf import _host_values


@pytest.mark.parametrize("ds", [torch.float64, torch.float32])
@pytest.mark.parametrize("de", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", [(), (1,)])
def test_host_values(ds, de, shape):
    sigma = torch.full(shape, 1.3, dtype=ds, requires_grad=True)
    ell = torch.tensor([0.1, 7.0, 1e-9], dtype=de, requires_grad=True)
    s, l = _host_values(sigma, ell)
    assert type(s) is float and s == float(sigma)
    assert l == [float(v) for v in ell]
