"""Images, gradients and optical depths of few and of shared rays against the
oracle: groups of 1 to 65 rays of one origin among lone rays (sums over the
wave, own atomics, partly filled waves), observers along axes and oblique
(axes a ray does not move along are left out), box, slab and sphere, one and
two lines, replayed and from the crossing lists.  Doubles: the same sums in
another order and with other roundings of the opacity's last operations, a
few hundred terms of relative error 2^-52 each, well inside 1e-10 of the
largest value (the bound of the other adjoint tests)."""
import numpy as np
import pytest

from paper_2001_11252_amd import workloads as W

pytestmark = pytest.mark.gpu

S = 0.6, 0.0, 0.8
T3 = tuple(np.full(3, 1.0 / np.sqrt(3.0)))


def _close(a, b):
    assert np.abs(a - b).max() <= 1e-10 * np.abs(b).max() + 1e-300


@pytest.mark.parametrize("group", [1, 3, 4, 5, 63, 64, 65])
@pytest.mark.parametrize("k,domain,two", [((0.0, 0.0, 1.0), "box", False), ((-1.0, 0.0, 0.0), "sphere", False),
                                          (S, "slab", True), (T3, "sphere", False), (T3, "box", True)])
def test_gradients_of_shared_and_lone_rays(orc, group, k, domain, two):
    from paper_2001_11252_amd import rmc
    rng = np.random.default_rng(group)
    s0 = lambda ln, T: orc.line_quantities(ln, T)["sigma0"]  # noqa: E731
    mesh = W.refined_mesh(2, 5, lambda lev, lo, hi: (np.abs(lo + hi - 1.0).max(axis=1) < 2.0 ** (2 - lev)))
    pb = W.static_sphere(s0, 20.0, 1e4, 1, level=0)
    pb.mesh = mesh
    n0 = pb.gas.n_hi[0]
    pb.gas = W.Gas(n0 * rng.lognormal(0.0, 0.5, mesh.n), np.full(mesh.n, 1e4) * rng.uniform(0.5, 2.0, mesh.n),
                   rng.normal(0.0, 1e6, (mesh.n, 3)), rng.uniform(0.0, 0.5, mesh.n) / mesh.box_cm)
    if domain == "box":
        pb.domain = W.Domain(W.DOM_BOX, (0.0, 0.0, 0.0, 0.0))
    elif domain == "slab":
        pb.domain = W.Domain(W.DOM_SLAB_Z, (0.5, 0.4, 0.0, 0.0))
    if two:
        pb.lines = [W.LYA, W.D_LYA]
    n_groups = 5
    orig = np.repeat(0.3 + 0.4 * rng.random((n_groups, 3)), group, axis=0)
    orig = np.concatenate([orig, 0.3 + 0.4 * rng.random((7, 3))])
    n = len(orig)
    x, w = rng.uniform(-6.0, 6.0, n), rng.random(n)
    G = rng.standard_normal((6, 6))
    pb.observers = [W.Observer(k, 6, 6, 1, (-1.0, 1.0, -1.0, 1.0), -1e30, 1e30)]
    img_o, gn_o, gk_o, gv_o = orc.raycast_image(pb, pb.observers[0], orig, x, w, G)
    ctx = rmc.Context.from_problem(pb, "fp64", sources=False)
    _close(ctx.raycast_image(0, orig, x, w), img_o)
    for g, go in zip(ctx.raycast_image_backward(0, orig, x, w, G), (gn_o, gk_o, gv_o)):
        _close(g, go)
    _close(ctx.raycast_image_tape(0, orig, x, w), img_o)
    for g, go in zip(ctx.raycast_image_backward_tape(G), (gn_o, gk_o, gv_o)):
        _close(g, go)
    d = rng.standard_normal((n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    _close(ctx.tau(orig, d, x), orc.tau(pb, orig, d, x))
    ctx.close()
