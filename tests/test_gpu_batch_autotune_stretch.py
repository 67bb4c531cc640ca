"""The batch tuner compares shapes on the same stretch of the run, two windows
of 8192 loop iterations here, also where launches are shorter than a slice.
A first problem's short walks leave the queue dry soon after the second's
packets, which walk past 8192 iterations and end before 16384, have started:
each shape's launch ends there, and the trial that follows has to go on until
they are done."""
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_trials_run_their_whole_stretch(prec):
    from paper_2001_11252_amd import rmc
    lanes = 256 * 64
    ctxs = []
    for n, events in ((lanes, 60), (2000, 10_000)):
        # at this depth all but a few packets stop at their event limit
        pb = W.static_sphere(rmc.sigma0, 1e7, 1e4, n, level=0)
        c = rmc.Context.from_problem(pb, prec)
        c.set_option(rmc.OPT_MAX_EVENTS, events)
        ctxs.append(c)
    ctxs[0].set_option(rmc.OPT_WAVES_PER_CU, 1)
    rmc.batch_autotune(ctxs, [1, 2], [lanes, 2000], trial_slices=1)
    # (the packets of the last shape tried, slices of 8192)
    assert (ctxs[0].get_packets(lanes)["status"] != 0).all()
    assert (ctxs[1].get_packets(2000)["status"] != 0).all()
    for c in ctxs:
        c.close()
