"""The hi+lo methods' plan of blocks and mode slices where the blocks' rounds decide: a launch of
narrow blocks that runs in one round keeps its modes whole."""
import pytest

from paper_2212_10961_amd import _lib as L
from test_fold_plan import _need, _tables


# (the second: 200 narrow blocks in one round; the third is split by either rule)
@pytest.mark.parametrize("shape,n,split", [((1500, 1200), 475, False), ((200, 200, 60), 475, False),
                                           ((1100, 900), 1500, True)])
def test_split_by_rounds(shape, n, split):
    cells = 1
    for s in shape:
        cells *= s
    need, tables = _need(n, shape, L.GRF_SEP_F16_X3), _tables(n, shape)
    assert (need > tables + cells) == split, (need, tables)
