"""Cubes of an observer alone (the ray-cast pass compiled for one observer),
among others and in a batch: the same rays, so the same deposits in another
order.  An element's sum of n deposits moves by up to n 2^-53 (2^-24 in float)
of itself; the elements here hold at most a few thousand in double and a few
hundred in float: 1e-10 and 1e-4 of the largest element.  Observers along axes
(axes a ray does not move along are left out) and oblique, one and two lines."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

DIRS = [(0.0, 0.0, 1.0), (-1.0, 0.0, 0.0), (0.6, 0.0, -0.8), tuple(np.full(3, 1.0 / np.sqrt(3.0)))]


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("two", [False, True])
def test_observer_alone_equals_among_others(orc, prec, tol, two):
    from paper_2001_11252_amd import rmc
    n = 3001
    pb = W.static_sphere(rmc.sigma0, 20.0, 1e4, n, level=0, tau_dust=0.5)
    n0, kd0 = pb.gas.n_hi[0], pb.gas.kappa_d[0]
    pb.mesh = W.refined_mesh(2, 5, lambda lev, lo, hi: (np.abs(lo + hi - 1.0).max(axis=1) < 2.0 ** (2 - lev)))
    rng = np.random.default_rng(3)
    m = pb.mesh.n
    pb.gas = W.Gas(n0 * rng.lognormal(0.0, 0.5, m), np.full(m, 1e4), rng.normal(0.0, 1e6, (m, 3)), np.full(m, kd0))
    if two:
        pb.lines = [W.LYA, W.D_LYA]
    obs = [W.Observer(k, 8, 8, 20, (-0.5, 0.5, -0.5, 0.5), -40.0, 40.0) for k in DIRS]

    def context(o):
        pb.observers = o
        return rmc.Context.from_problem(pb, prec)

    ctx = context(obs)
    all_st = ctx.run(11, 0, n)
    ref = [ctx.get_cube(i) for i in range(len(obs))]
    cs = [context([o]) for o in obs]
    st = [c.run(11, 0, n) for c in cs]
    assert sum(s["peel_rays"] for s in st) == all_st["peel_rays"] > 4 * n
    for c, r in zip(cs, ref):
        assert r.max() > 0.0
        assert np.abs(c.get_cube(0) - r).max() <= tol * r.max()
        c.reset_cubes()
    rmc.batch_run(cs, [11] * len(cs), [n] * len(cs))
    for c, r in zip(cs, ref):
        assert np.abs(c.get_cube(0) - r).max() <= tol * r.max()
