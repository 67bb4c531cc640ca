"""The kernels compiled for two lines against those for four: two more lines
of no abundance add nothing to any opacity, so the packets are the same bit
for bit (bulk kernel, walkers, batches, queued peel-off)."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("compact", [0, 1])
@pytest.mark.parametrize("model", ["deuterium", "wind"])
def test_two_line_kernels_equal_the_four_line_ones(prec, compact, model):
    from paper_2001_11252_amd import rmc
    n = 3001
    out = []
    for extra in (0, 2):
        if model == "wind":
            pb = W.feii_wind(rmc.sigma0, n, level=3)
        else:
            pb = W.deuterium_sphere(rmc.sigma0, n, N_HI=30.0 / rmc.sigma0(W.LYA, 1e4), d_to_h=0.05)
            pb.observers = [W.Observer((0.0, 0.0, 1.0), 5, 4, 6, (-0.3, 0.5, -0.5, 0.5), -3.0, 9.0)]
        pb.lines = list(pb.lines) + [replace(ln, abundance=0.0, fluor=()) for ln in (W.MGII_2796, W.MGII_2804)][:extra]
        ctxs = [rmc.Context.from_problem(pb, prec) for _ in range(2)]
        for c in ctxs:
            c.set_option(rmc.OPT_COMPACT, compact)
        st = [ctxs[0].run(3, 0, n)]
        pk = [ctxs[0].get_packets()]
        per, _ = rmc.batch_run(ctxs, [3, 4], [n, 77])
        out.append((st + per, pk + [ctxs[0].get_packets(), ctxs[1].get_packets()]))
        for c in ctxs:
            c.close()
    for a, b in zip(out[0][0], out[1][0]):
        for k in ("emitted", "escaped", "scatterings", "crossings", "peel_rays", "peel_crossings", "peel_dropped"):
            assert a[k] == b[k], k
    for a, b in zip(out[0][1], out[1][1]):
        for k in a:
            assert np.array_equal(a[k], b[k]), k
