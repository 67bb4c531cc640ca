"""FP32 gradients of rays that share waves: the sum of those of each ray run
alone, which adds its own terms without any sum over the wave.  The terms are
the same floats taken to double; only the order of a leaf's additions
differs, at most 2 N 2^-53 of the sum of the N terms' magnitudes (here below
1e-11 of the sum over rays of each gradient's magnitude).  Groups of rays of
one origin among lone ones (sums over the wave, own atomics, partly filled
waves), one and two lines, replayed and from the crossing lists."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [1, 3, 4, 63, 64, 65])
@pytest.mark.parametrize("k,two", [((0.0, 0.0, 1.0), False), ((0.6, 0.0, 0.8), True)])
def test_float_gradients_are_the_sums_over_lone_rays(group, k, two):
    from paper_2001_11252_amd import rmc
    rng = np.random.default_rng(group)
    mesh = W.refined_mesh(2, 4, lambda lev, lo, hi: (np.abs(lo + hi - 1.0).max(axis=1) < 2.0 ** (2 - lev)))
    pb = W.static_sphere(rmc.sigma0, 20.0, 1e4, 1, level=0)
    n0 = pb.gas.n_hi[0]
    pb.mesh = mesh
    pb.gas = W.Gas(n0 * rng.lognormal(0.0, 0.5, mesh.n), np.full(mesh.n, 1e4) * rng.uniform(0.5, 2.0, mesh.n),
                   rng.normal(0.0, 1e6, (mesh.n, 3)), rng.uniform(0.0, 0.5, mesh.n) / mesh.box_cm)
    if two:
        pb.lines = [W.LYA, W.D_LYA]
    orig = np.concatenate([np.repeat(0.3 + 0.4 * rng.random((3, 3)), group, axis=0), 0.3 + 0.4 * rng.random((7, 3))])
    n = len(orig)
    x, w, G = rng.uniform(-6.0, 6.0, n), rng.random(n), rng.standard_normal((6, 6))
    pb.observers = [W.Observer(k, 6, 6, 1, (-1.0, 1.0, -1.0, 1.0), -1e30, 1e30)]
    ctx = rmc.Context.from_problem(pb, "fp32", sources=False)
    lone = [ctx.raycast_image_backward(0, orig[i:i + 1], x[i:i + 1], w[i:i + 1], G) for i in range(n)]
    replayed = ctx.raycast_image_backward(0, orig, x, w, G)
    ctx.raycast_image_tape(0, orig, x, w)
    listed = ctx.raycast_image_backward_tape(G)
    ctx.close()
    for j in range(3):
        total, size = sum(g[j] for g in lone), sum(np.abs(g[j]) for g in lone)
        assert size.max() > 0.0
        assert (np.abs(replayed[j] - total) <= 1e-11 * size).all(), j
        # (the lists keep segments as floats: two roundings of 2^-24 a term)
        assert (np.abs(listed[j] - total) <= 2.0 ** -22 * size).all(), j
