"""The workspace of the hi+lo methods, which shows whether their mode split is planned: no split
where its sums' passes cost more than the stages they save, one where they save much."""
import ctypes

import pytest

from paper_2212_10961_amd import _lib as L


def _need(n, shape, method):
    m = L.GrfModes()
    m.dim, m.n, m.sigma = len(shape), n, 1.0
    m.ell = (ctypes.c_double * 3)(1.0, 1.0, 1.0)
    m.z = m.phi = 16
    g = L.GrfGrid()
    g.n = (ctypes.c_int64 * 3)(*(tuple(shape) + (1,))[:3])
    g.h = (ctypes.c_double * 3)(1.0, 1.0, 1.0)
    b = ctypes.c_size_t()
    assert L.load().eval_field_grid_ws_size(ctypes.byref(m), ctypes.byref(g), method, ctypes.byref(b)) == 0
    return b.value


def _tables(n, shape):
    # (nx + ny) hi+lo entries of 8 bytes per mode, in 3-D with nz of 8 bytes
    return (n + 63) // 64 * 64 * 8 * sum(shape)


@pytest.mark.parametrize("shape,n,split", [((256, 256, 64), 256, False), ((2048, 2048), 256, False),
                                           ((150, 97, 21), 700, True), ((203, 171, 85), 3000, True),
                                           ((256, 256), 2048, True)])
def test_split_where_it_pays(shape, n, split):
    cells = 1
    for s in shape:
        cells *= s
    need, tables = _need(n, shape, L.GRF_SEP_F16_X3), _tables(n, shape)
    assert (need > tables + cells) == split, (need, tables)
