"""The deferred peel-off queue against the inline walk, at the numbers of
transport waves (queue regions) where the index of its jobs turns: one
region, one lane group of 64 and one more, one block tile of 1024 and one
more, beyond 64 x 64.  Each ray is walked once or the counts of leaves
crossed and of deposits outside the cube would differ; they are whole
numbers and equal."""
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [1, 2, 63, 64, 65, 1024, 1025, 4097])
def test_every_queued_ray_is_walked_once(waves):
    from paper_2001_11252_amd import rmc
    n = 64 * waves - 7
    pb = W.static_sphere(rmc.sigma0, 20.0, 1e4, n, level=2, tau_dust=0.3)
    pb.observers = [W.Observer((0.0, 0.0, 1.0), 6, 5, 11, (-0.3, 0.5, -0.5, 0.5), -2.0, 8.0),
                    W.Observer((1.0, 0.0, 0.0), 4, 4, 7, (-0.5, 0.5, -0.5, 0.5), -8.0, 8.0)]
    out = {}
    for defer in (0, 1):
        c = rmc.Context.from_problem(pb, "fp64")
        c.set_option(rmc.OPT_BLOCK, 64)
        c.set_option(rmc.OPT_WAVES_PER_CU, 32)
        c.set_option(rmc.OPT_MAX_EVENTS, 4)
        c.set_option(rmc.OPT_PEEL_DEFER, defer)
        st = c.run(9, 0, n)
        out[defer] = st
        c.close()
    for k in ("emitted", "scatterings", "peel_rays", "peel_crossings", "peel_dropped"):
        assert out[0][k] == out[1][k], k
    assert out[1]["peel_dropped"] > 0 and out[1]["peel_deferred"] > 0.1 * out[1]["peel_rays"]
