"""Room of the deferred peel-off queue: once a first run has enlarged it, float
runs of several observers and runs in long slices end no launch early for want
of room (they queue several times the rays a launch of one observer does)."""
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

S3 = 3.0 ** -0.5


@pytest.mark.parametrize("observers,slice_iters,tau0,max_events", [(3, 2048, 2e3, 0), (1, 8192, 5e3, 8000)])
def test_the_queue_holds_a_slice_of_rays(observers, slice_iters, tau0, max_events):
    from paper_2001_11252_amd import rmc
    n = 400_000
    pb = W.c2_dusty_sphere(rmc.sigma0, n, tau0)
    pb.observers = [W.Observer(k, 16, 16, 10, (-0.5, 0.5, -0.5, 0.5), -60.0, 60.0)
                    for k in ((0.0, 0.0, 1.0), (1.0, 0.0, 0.0), (S3, S3, S3))[:observers]]
    c = rmc.Context.from_problem(pb, "fp32")
    c.set_option(rmc.OPT_SLICE_ITERS, slice_iters)
    c.set_option(rmc.OPT_MAX_EVENTS, max_events)
    c.run(5, 0, n)
    st = c.run(5, 0, n)
    c.close()
    assert st["emitted"] == n
    assert st["slices_cut"] == 0
