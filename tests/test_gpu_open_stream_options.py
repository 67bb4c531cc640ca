"""Options set while a stream is open hold from the next begin on: the open
stream keeps the launch shape, the slots, reserves and queue regions and the
form of the scattering draw it began with.  Each option is changed after the
begin and changed back after the first step; packets, counts and the steps'
ends are those of a stream left alone, bit for bit."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = ("emitted", "escaped", "absorbed", "stuck", "scatterings", "dust_scatterings", "crossings", "peel_rays",
          "peel_crossings", "peel_dropped")
# option, its value at the begin, its value from then on, other options
CHANGES = [
    ("BLOCK", 64, 256, {}),
    ("BLOCK", 64, 256, {"COMPACT": 0}),
    ("BLOCK", 256, 64, {"WAVES_PER_CU": 1}),
    ("COMPACT", 0, 1, {}),
    ("COMPACT", 0, 1, {"BLOCK": 64, "WAVES_PER_CU": 1, "SLICE_ITERS": 40}),
    ("COMPACT", 1, 0, {}),
    ("REGROUP", 1, 0, {"COMPACT": 0, "SLICE_ITERS": 3}),
    ("REGROUP", 1, 0, {"WAVES_PER_CU": 1, "SLICE_ITERS": 3}),
    ("REGROUP", 0, 1, {"COMPACT": 0, "SLICE_ITERS": 3}),
    ("REFILL", 1, 64, {"WAVES_PER_CU": 1}),
    ("SLICE_ITERS", 7, 2048, {"COMPACT": 0}),
    ("SLICE_ITERS", 7, 1, {}),
    ("WAVES_PER_CU", 1, 8, {}),
    ("PEEL_DEFER", 1, 0, {}),
    ("PEEL_DEFER", 0, 1, {}),
    ("MAX_EVENTS", 50, 9, {}),
    ("FORWARD_ONLY", 0, 1, {"MAX_EVENTS": 50}),
]


def _run(rmc, pb, prec, n, option, at_begin, later, others):
    c = rmc.Context.from_problem(pb, prec)
    opt = getattr(rmc, "OPT_" + option)
    for k, v in others.items():
        c.set_option(getattr(rmc, "OPT_" + k), v)
    c.set_option(opt, at_begin)
    c.stream_begin(11, 0, n)
    ends = []
    while True:
        if later is not None:
            c.set_option(opt, later if len(ends) != 1 else at_begin)
        sl, rem = c.stream_step()
        ends.append(sl["emitted"])
        if rem == 0:
            break
    st = c.stream_end()
    pk = c.get_packets()
    c.close()
    return st, pk, ends


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [9001, 40001])
@pytest.mark.parametrize("option,at_begin,later,others", CHANGES)
def test_open_stream_keeps_the_options_of_its_begin(prec, n, option, at_begin, later, others):
    from paper_2001_11252_amd import rmc
    pb = W.static_sphere(rmc.sigma0, 15.0, 1e4, n, level=2, tau_dust=0.4)
    pb.observers = [W.Observer((0.6, 0.0, 0.8), 5, 4, 6, (-0.3, 0.5, -0.5, 0.5), -3.0, 9.0)]
    st0, pk0, ends0 = _run(rmc, pb, prec, n, option, at_begin, None, others)
    st, pk, ends = _run(rmc, pb, prec, n, option, at_begin, later, others)
    for k in pk0:
        assert np.array_equal(pk[k], pk0[k]), k
    for k in COUNTS:
        assert st[k] == st0[k], k
    assert sum(ends) == n
    if "WAVES_PER_CU" not in others and option != "WAVES_PER_CU":   # every packet starts in the first step
        assert ends == ends0
