"""The work queue of the transport: whatever the launch shape (waves, slice
length, refill threshold, reserves taken while the queue is long), every
packet is run once and gives the same bits.  256 waves of one block each
take reserves beyond their need while more than 32768 packets remain."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(rmc, pb, prec, n, block, waves, slice_iters, refill, seed=5):
    c = rmc.Context.from_problem(pb, prec)
    for o, v in ((rmc.OPT_BLOCK, block), (rmc.OPT_WAVES_PER_CU, waves), (rmc.OPT_SLICE_ITERS, slice_iters),
                 (rmc.OPT_REFILL, refill)):
        c.set_option(o, v)
    st, pk = c.run(seed, 0, n), c.get_packets()
    c.close()
    return st, pk


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 64, 65, 16384, 49153, 200_003])
def test_every_packet_runs_once_in_any_launch_shape(prec, n):
    from paper_2001_11252_amd import rmc
    pb = W.static_sphere(rmc.sigma0, 2.0, 1e4, n, level=2, tau_dust=0.4)
    st0, p0 = _run(rmc, pb, prec, n, 256, 0, 2048, 1)
    assert st0["emitted"] == n and (p0["status"] != 0).all()
    assert st0["escaped"] == (p0["status"] == 1).sum() and st0["absorbed"] == (p0["status"] == 2).sum()
    for block, waves, sl, refill in ((64, 1, 5, 1), (64, 1, 2048, 48), (128, 4, 1, 64)):
        st, pk = _run(rmc, pb, prec, n, block, waves, sl, refill)
        for k in p0:
            assert np.array_equal(p0[k], pk[k]), (k, block, waves, sl)
        for k in ("emitted", "escaped", "absorbed", "stuck", "scatterings", "dust_scatterings", "crossings"):
            assert st0[k] == st[k], k
