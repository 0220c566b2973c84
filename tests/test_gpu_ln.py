"""The kernels' logarithm (ln.h), seen through alpha_s: knots that lie on a line in
ln Q^2 are interpolated by that line, so alpha_s(Q^2) = ln Q^2."""
import math

import numpy as np
import pytest

from helpers import cfg0_grid
from paper_2012_08221_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_08221_amd import api as a
    return a


@pytest.mark.parametrize("lo,hi", [(1e-9, 1.0), (1.0, 1e10), (0.5, 2.0), (0.999, 1.001),
                                   (2.0 ** -0.5, 2.0 ** 0.5), (1e-300, 1e300), (5e-324, 1e-307)])
def test_ln_over_every_range(api, lo, hi):
    """Powers of two, sqrt(1/2) times them (where the reduction turns) and their
    neighbours among random points.  Tolerance: the logarithm within an ulp of the
    largest, and as much again for each of the coordinate, the four weights' products
    and the knots themselves."""
    g = cfg0_grid()
    knots = np.geomspace(max(lo, 5e-324), hi, 9)
    knots[0], knots[-1] = lo, hi
    logs = np.log(knots)
    pdf = api.mkPDF(wl.GridSpec(pids=g.pids, x=g.x, q2=g.q2, q_off=g.q_off, xf=g.xf,
                                as_q2=knots, as_val=logs))
    rng = np.random.default_rng(int(abs(math.log(lo))))
    q2 = np.exp(rng.uniform(logs[0], logs[-1], 20000))
    two = np.ldexp(1.0, np.arange(-1074, 1023))
    for t in (two, two * math.sqrt(0.5)):
        q2 = np.concatenate([q2, t, np.nextafter(t, 0.0), np.nextafter(t, np.inf)])
    q2 = q2[(q2 >= lo) & (q2 <= hi)]
    got = pdf.alphasQ2(q2).cpu().numpy()
    big = np.abs(logs).max()
    assert np.abs(got - np.log(q2)).max() <= 7 * np.spacing(big)
