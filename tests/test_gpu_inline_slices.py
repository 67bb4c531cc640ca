"""Runs that walk their peel-off rays inline (RMC_OPT_PEEL_DEFER = 0) launch
whole slices, also when the queue of packets runs dry in one: no walkers
follow, and packets spread over the lanes walk faster than gathered.  Walks
of 700 events, one lane's worth and then some: the second packets start in the
middle of the first slice of 2048 passes and end in it."""
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

LANES = 256 * 64


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("compact", [0, 1])
def test_inline_slices_are_whole(prec, compact):
    from paper_2001_11252_amd import rmc
    n = LANES + 3001
    pb = W.static_sphere(rmc.sigma0, 1e6, 1e4, n, level=1)
    pb.observers = [W.Observer((0.0, 0.0, 1.0), 8, 8, 10, (-0.5, 0.5, -0.5, 0.5), -60.0, 60.0)]
    c = rmc.Context.from_problem(pb, prec)
    for o, v in ((rmc.OPT_PEEL_DEFER, 0), (rmc.OPT_BLOCK, 64), (rmc.OPT_WAVES_PER_CU, 1), (rmc.OPT_MAX_EVENTS, 700),
                 (rmc.OPT_COMPACT, compact), (rmc.OPT_SLICE_ITERS, 2048)):
        c.set_option(o, v)
    c.stream_begin(7, 0, n)
    sl, left = c.stream_step()
    st = c.stream_end()
    c.close()
    assert left == 0 and sl["emitted"] == n and st["emitted"] == n
