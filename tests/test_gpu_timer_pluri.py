"""The kernel timer of a bitruncated grid: one pair per call, and where the modes are split it covers
the pass that adds the slices (and makes the rule)."""
import numpy as np
import pytest
import torch

from paper_2212_10961_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_10961_amd.grf as g
    return g


def _pair(grf, dim, n):
    ell = (9.0, 7.0, 3.0)[:dim]
    return [grf.modes_from_tables(*grf.make_modes(dim, c, n, s), 1.0, ell) for c, s in ((wl.GAUSSIAN, 5), (wl.EXPONENTIAL, 6))]


def _rule(grf):
    return grf.trunc2([0.0], [0.0], np.arange(4, dtype=np.uint8).reshape(2, 2), np.arange(4, dtype=np.float32))


def _ms(grf, run, calls):
    run()
    torch.cuda.synchronize()
    with grf.KernelTimer() as kt:
        for _ in range(calls):
            run()
        torch.cuda.synchronize()
    ms, n = kt.read()
    assert n == calls
    return ms / calls


# split and unsplit, one-pass and hi+lo
@pytest.mark.parametrize("meth", ["sep_f16", "sep_f16_x3", "sep_bf16_x3"])
@pytest.mark.parametrize("shape,n", [((96, 64), 64), ((300, 200), 2000), ((256, 256, 64), 64), ((40, 30, 20), 2000)])
def test_one_pair_per_call(grf, shape, n, meth):
    print(f"case pluri timer {shape} n={n} {meth}", flush=True)
    m1, m2 = _pair(grf, len(shape), n)
    assert 0.0 < _ms(grf, lambda: grf.pluri_grid(m1, m2, shape, _rule(grf), method=meth), 3) < 1e2


def test_split_covers_the_slice_pass(grf):
    """240 blocks of 128 x 128 cells split 256 modes in two.  The same contraction with a second pass
    that stores 13 bytes more per cell has to take longer by the timer (best of six)."""
    shape, n = (1900, 2048), 256
    m1, m2 = _pair(grf, 2, n)
    rule = _rule(grf)
    C = shape[0] * shape[1]
    few = {"facies": torch.empty(C, dtype=torch.uint8, device="cuda")}
    many = dict(few, **{k: torch.empty(C, device="cuda") for k in ("value", "y1", "y2")})

    def run(out, **kw):
        return lambda: grf.pluri_grid(m1, m2, shape, rule, method="sep_f16", out=out, **kw)

    t = [(_ms(grf, run(few), 10), _ms(grf, run(many, want_value=True, keep_fields=True), 10)) for _ in range(6)]
    a, b = (min(v) * 1e3 for v in zip(*t))
    print(f"  facies {a:.1f} us, facies, values and fields {b:.1f} us", flush=True)
    assert b > 1.04 * a
