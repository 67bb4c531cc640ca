"""Launches that end because the queue ran dry in them: more packets than
lanes, the last ones starting in the middle of a launch.  Every packet is run
once and gives the bits of a run whose lanes start all packets at once, with
one, a few and a lane's worth of packets left over, and with walks that end
before and after the second look at the queue (511 iterations)."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

LANES = 256 * 64


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("extra", [1, 65, 3001, LANES])
@pytest.mark.parametrize("max_events", [200, 700])
def test_packets_left_over_when_the_queue_runs_dry(prec, extra, max_events):
    from paper_2001_11252_amd import rmc
    n = LANES + extra
    pb = W.static_sphere(rmc.sigma0, 1e5, 1e4, n, level=2, tau_dust=0.4)
    pb.observers = [W.Observer((0.0, 0.0, 1.0), 8, 8, 10, (-0.5, 0.5, -0.5, 0.5), -60.0, 60.0)]
    out = []
    for waves in (0, 1):   # all packets at once; one wave a CU
        c = rmc.Context.from_problem(pb, prec)
        c.set_option(rmc.OPT_MAX_EVENTS, max_events)
        if waves:
            c.set_option(rmc.OPT_BLOCK, 64)
            c.set_option(rmc.OPT_WAVES_PER_CU, waves)
        out.append((c.run(7, 0, n), c.get_packets()))
        c.close()
    (st0, p0), (st1, p1) = out
    assert st0["emitted"] == n and (p0["status"] != 0).all()
    for k in p0:
        assert np.array_equal(p0[k], p1[k]), k
    for k in ("emitted", "escaped", "absorbed", "stuck", "scatterings", "dust_scatterings", "crossings", "peel_rays"):
        assert st0[k] == st1[k], k
