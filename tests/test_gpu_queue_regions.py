"""The deferred peel-off queue where its regions belong to k_transport's waves
alone (RMC_OPT_COMPACT = 0: no walkers), at the counts where the index of its
jobs turns (k_peel_scan, region_of): one region, one lane group of 64 and one
more, one block tile of 1024 and one more, beyond 64 x 64; and with gathered
packets too many for the walkers, which k_transport runs in half slices over
fewer regions than the full grid has.  Whole-number counts are equal; a cube
element's FP64 sum of N deposits depends on their order by at most
2 N 2^-53 of it."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = ("emitted", "escaped", "absorbed", "stuck", "scatterings", "dust_scatterings", "crossings", "peel_rays",
          "peel_crossings", "peel_dropped")
OBSERVERS = [W.Observer((0.0, 0.0, 1.0), 6, 5, 11, (-0.3, 0.5, -0.5, 0.5), -2.0, 8.0),
             W.Observer((0.6, 0.0, 0.8), 4, 4, 7, (-0.5, 0.5, -0.5, 0.5), -8.0, 8.0)]


@pytest.mark.parametrize("waves", [1, 2, 63, 64, 65, 1024, 1025, 4097])
def test_every_queued_ray_is_walked_once_without_walkers(waves):
    from paper_2001_11252_amd import rmc
    n = 64 * waves - 7
    pb = W.static_sphere(rmc.sigma0, 20.0, 1e4, n, level=2, tau_dust=0.3)
    pb.observers = OBSERVERS
    out = {}
    for defer in (0, 1):
        c = rmc.Context.from_problem(pb, "fp64")
        for o, v in ((rmc.OPT_BLOCK, 64), (rmc.OPT_WAVES_PER_CU, 32), (rmc.OPT_MAX_EVENTS, 4), (rmc.OPT_COMPACT, 0),
                     (rmc.OPT_PEEL_DEFER, defer)):
            c.set_option(o, v)
        out[defer] = c.run(9, 0, n)
        c.close()
    for k in COUNTS:
        assert out[0][k] == out[1][k], k
    assert out[1]["peel_dropped"] > 0 and out[1]["peel_deferred"] > 0.1 * out[1]["peel_rays"]


# beyond the walkers' largest count (64 x 1024 in double, 32 x 1024 in float)
@pytest.mark.parametrize("prec,n,walkers", [("fp32", 100_003, 32768), ("fp64", 131_072, 65536)])
def test_gathered_transport_with_a_queue(prec, n, walkers):
    from paper_2001_11252_amd import rmc
    pb = W.static_sphere(rmc.sigma0, 30.0, 1e4, n, level=2, tau_dust=0.3)
    pb.observers = OBSERVERS
    out = []
    for compact in (0, 1):
        c = rmc.Context.from_problem(pb, prec)
        c.set_option(rmc.OPT_COMPACT, compact)
        c.set_option(rmc.OPT_SLICE_ITERS, 8)
        c.stream_begin(3, 0, n)
        left = []
        while not left or left[-1]:
            left.append(c.stream_step()[1])
        st = c.stream_end()
        out.append((st, c.get_packets(), [c.get_cube(o) for o in range(2)], left))
        c.close()
    (s0, p0, c0, l0), (s1, p1, c1, l1) = out
    # packets left after a step: few enough to gather, too many for the walkers; the
    # next launch runs half a slice
    i = next(i for i, r in enumerate(l1) if r <= 3 * n // 4)
    assert l1[:i + 1] == l0[:i + 1] and l1[i] > walkers and l1[i + 1] > l0[i + 1]
    for k in p0:
        assert np.array_equal(p0[k], p1[k]), k
    for k in COUNTS + ("peel_deferred",):
        assert s0[k] == s1[k], k
    assert s1["peel_deferred"] > 0
    for a, b in zip(c0, c1):
        assert a.sum() > 0
        if prec == "fp64":
            assert (np.abs(a - b) <= 2 * s0["peel_deferred"] * 2.0 ** -53 * a).all()
