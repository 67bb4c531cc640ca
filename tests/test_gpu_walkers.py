"""The last packets' kernel (P packets a wave, draws and peel-off by all its
lanes) against the bulk kernel (RMC_OPT_COMPACT = 0): the same packets bit for
bit and the same counts, at packet counts where the packets per wave change
(1 to 64, partly filled last waves), with events left pending by a regrouped
launch, two lines, fluorescence, dust, observers, core-skipping, and batches
whose problems must not share a wave."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = ("emitted", "escaped", "absorbed", "stuck", "scatterings", "dust_scatterings", "crossings", "peel_rays",
          "peel_crossings", "peel_dropped")


def _problem(rmc, model, n):
    if model == "dust":
        pb = W.static_sphere(rmc.sigma0, 15.0, 1e4, n, level=2, tau_dust=0.4)
    elif model == "two_lines":
        pb = W.deuterium_sphere(rmc.sigma0, n, N_HI=20.0 / rmc.sigma0(W.LYA, 1e4), d_to_h=0.05)
    elif model == "fluorescence":
        return W.feii_wind(rmc.sigma0, n, level=3)
    else:
        pb = W.thick_sphere(rmc.sigma0, n, 3e4)
    pb.observers = [W.Observer(k, 5, 4, 6, (-0.3, 0.5, -0.5, 0.5), -3.0, 9.0) for k in ((0.0, 0.0, 1.0), (0.6, 0.0, 0.8))]
    return pb


def _run(rmc, pb, prec, n, compact, model, **opts):
    c = rmc.Context.from_problem(pb, prec)
    c.set_option(rmc.OPT_COMPACT, compact)
    for k, v in opts.items():
        c.set_option(getattr(rmc, "OPT_" + k), v)
    if model == "skip":
        c.set_core_skip(1.0, 0.2)
        c.set_option(rmc.OPT_MAX_EVENTS, 40)
    st, pk = c.run(21, 0, n), c.get_packets()
    c.close()
    return st, pk


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("model", ["dust", "two_lines", "fluorescence", "skip"])
@pytest.mark.parametrize("n", [1, 63, 257, 2049, 9001, 65535])
def test_same_packets_as_the_bulk_kernel(prec, model, n):
    from paper_2001_11252_amd import rmc
    pb = _problem(rmc, model, n)
    ref = _run(rmc, pb, prec, n, 0, model)
    for opts in ({}, {"SLICE_ITERS": 3}, {"REGROUP": 1, "SLICE_ITERS": 2, "WAVES_PER_CU": 1}):
        st, pk = _run(rmc, pb, prec, n, 1, model, **opts)
        for k in pk:
            assert np.array_equal(pk[k], ref[1][k]), (k, opts)
        for k in COUNTS:
            assert st[k] == ref[0][k], (k, opts)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes", [(1, 1, 1), (3, 700, 64, 1, 0, 129), (40, 30, 900, 5000, 8, 33000)])
def test_batch_packets_equal_single_runs(prec, sizes):
    from paper_2001_11252_amd import rmc
    models = ["dust", "two_lines", "dust", "fluorescence", "two_lines", "dust"]
    pbs = [_problem(rmc, m, max(n, 1)) for m, n in zip(models, sizes)]
    ctxs = [rmc.Context.from_problem(p, prec) for p in pbs]
    per, tot = rmc.batch_run(ctxs, list(range(5, 5 + len(sizes))), list(sizes))
    assert tot["emitted"] == sum(sizes)
    for i, (pb, n) in enumerate(zip(pbs, sizes)):
        if n == 0:
            continue
        got = ctxs[i].get_packets(n)
        c = rmc.Context.from_problem(pb, prec)
        c.set_option(rmc.OPT_COMPACT, 0)
        st = c.run(5 + i, 0, n)
        ref = c.get_packets()
        c.close()
        for k in ref:
            assert np.array_equal(got[k], ref[k]), (k, i)
        for k in COUNTS:
            assert per[i][k] == st[k], (k, i)
    for c in ctxs:
        c.close()
