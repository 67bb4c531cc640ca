"""Spectra against the counts of the same packets on the host, exactly: one bin
and many, the most bins a block counts by itself and one more, one packet, a
partly filled block and more packets than one sweep of the grid takes."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 257, 300_001])
def test_spectrum_counts_every_escaped_packet(orc, n):
    from paper_2001_11252_amd import rmc
    pb = W.static_sphere(rmc.sigma0, 0.5, 1e4, n, level=1, tau_dust=0.5)
    ctx = rmc.Context.from_problem(pb, "fp32")
    ctx.run(5, 0, n)
    pk = ctx.get_packets()
    x = pk["x"][pk["status"] == 1]
    for nbins, lo, hi in ((1, -50.0, 50.0), (700, -2.0, 1.5), (8192, -6.0, 6.0), (8193, -6.0, 6.0)):
        fb = (x - lo) / (hi - lo) * nbins
        b = np.floor(fb[(fb >= 0.0) & (fb < nbins)]).astype(np.int64)
        assert np.array_equal(ctx.get_spectrum(nbins, lo, hi), np.bincount(b, minlength=nbins).astype(np.float64))
