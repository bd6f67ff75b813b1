"""Sets of few large spheres: the link pass cuts the planes around a sphere into more slabs, from
a radius of 15 on, as the room of the set says (max_radius), up to 64.  State against the oracle
on both sides of each rule; and the time of the link pass beside the fluid kernel's, which does
not grow with the radius as the eight waves of one workgroup would.  The re-projection of a large sphere that
hardly moves searches for changed nodes only once it may have reached one: against the oracle
where it slows down, turns and comes back, and where another sphere runs into it; and its time."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _sets(shape, x, r, v, w, max_radius, bc, precision="fp64", **kw):
    from paper_1808_08921_amd.lbdem import LatticeSet

    params = dict(nx=shape[0], ny=shape[1], nz=shape[2], tau=0.8, rho_f=1.0, bc=bc, rho_p=3.0, E=5.0, nu=0.2, mu=0.3,
                  max_particles=len(r), max_radius=max_radius)
    gs = LatticeSet([params], precision=precision, graph_steps=3, **kw)
    gs.particles_set(0, x, r, v=v, w=w)
    s = oracle.Sim(*shape, tau=0.8, bc=bc, E=5.0, nu=0.2, mu=0.3, rho_p=3.0)
    s.set_particles(x, r, v=v, w=w)
    return gs, s


@pytest.mark.parametrize("node_lists", [0, 2])
@pytest.mark.parametrize("shape,r,max_radius,bc", [
    ((36, 38, 37), 14.4, 14.4, (0,) * 6),   # 40 planes: 8 slabs
    ((36, 38, 37), 14.4, 14.6, (0,) * 6),   # 41 planes: 16
    ((44, 42, 43), 18.7, 19.0, (0,) * 6),   # 16 slabs, a narrow lattice
    ((30, 29, 31), 6.3, 34.6, (1,) * 6),    # 32 slabs of which most hold nothing
    ((30, 29, 31), 6.3, 90.0, (1,) * 6),    # 64 slabs
    ((30, 29, 31), 6.3, 90.0, (0,) * 6),    # 64 slabs, two images a node
])
def test_state_matches_the_oracle(shape, r, max_radius, bc, node_lists):
    x = np.array([[0.5 * n - 0.3 for n in shape]])
    v, w = np.array([[0.03, -0.02, 0.05]]), np.array([[0.001, 0.002, -0.001]])
    gs, s = _sets(shape, x, np.array([r]), v, w, max_radius, bc, node_lists=node_lists)
    try:
        for n in (1, 2, 9):
            gs.step(n)
            s.step(n)
            got, want = gs.particles_get(0), s.particles()
            assert np.array_equal(gs.owner(0), s.owner())
            for k in ("x", "v", "w", "force", "torque"):
                assert np.abs(got[k] - want[k]).max() <= 1e-10 * max(np.abs(want[k]).max(), 1e-3), k
        assert gs.status() & 0x1da == 0
    finally:
        gs.close()
        s.close()


def test_link_pass_of_one_large_sphere():
    """A sphere of radius 60 at rest in 160^3 nodes: the link pass and the motion together take
    less than one and a half times as long as the fluid kernel."""
    from paper_1808_08921_amd.lbdem import LatticeSet

    params = dict(nx=160, ny=160, nz=160, tau=0.8, rho_f=1.0, bc=(0,) * 6, rho_p=5000.0, max_particles=1,
                  max_radius=60.0)
    with LatticeSet([params], precision="fp32") as gs:
        gs.particles_set(0, [[80.3, 79.8, 80.1]], [60.0])
        gs.step(20)
        gs.timing_enable()
        gs.step(20)
        links, motion, fluid, _, _ = gs.timing_read()[0]
    assert links + motion < 1.5 * fluid


def _pair(params, x, r, **state):
    """The set, the same set with room for more particles than its lattices have nodes, which has
    no place to keep what the watch needs and searches in every step, and the oracle."""
    from paper_1808_08921_amd.lbdem import LatticeSet

    room = dict(nx=1, ny=1, nz=1, bc=(1,) * 6, max_particles=8191, max_radius=params["max_radius"])
    more = params["nx"] * params["ny"] * params["nz"] // 8191 + 1
    lists = params.pop("node_lists")
    sets = [LatticeSet([params] + [room] * n, precision="fp64", graph_steps=0, node_lists=lists) for n in (0, more)]
    for gs in sets:
        gs.particles_set(0, x, r, **state)
    s = oracle.Sim(params["nx"], params["ny"], params["nz"], tau=params["tau"], bc=params["bc"], rho_p=params["rho_p"],
                   E=params["E"], nu=params["nu"], mu=0.0)
    s.set_rest_free(bool(params.get("rest_free")))
    s.set_particles(x, r, **state)
    return sets + [s]


def _follow(gs, ref, s, steps, every):
    for _ in range(0, steps, every):
        for one in (gs, ref, s):
            one.step(every)
        own = gs.owner(0)
        assert np.array_equal(own, s.owner()) and np.array_equal(own, ref.owner(0))
        got, want = gs.particles_get(0), ref.particles_get(0)
        for k in got:
            assert np.array_equal(got[k], want[k]), k
    assert gs.status() & 0x1da == 0


@pytest.mark.parametrize("node_lists", [0, 2])
def test_large_sphere_that_turns(node_lists):
    """From 2e-4 a step to rest and back, over seven nodes of its surface and back,
    with a checkpoint on the way."""
    rho_p, r, a = 50.0, 13.0, -2e-6
    x, v = np.array([[15.37, 15.81, 16.43]]), np.array([[2e-4, 1e-5, -3e-5]])
    fg = np.array([[a * rho_p * 4.0 / 3.0 * np.pi * r ** 3, 0.0, 0.0]])
    params = dict(nx=31, ny=32, nz=33, tau=0.8, rho_f=1.0, bc=(0,) * 6, rho_p=rho_p, E=10.0, nu=0.2, max_particles=1,
                  max_radius=r, node_lists=node_lists)
    gs, ref, s = _pair(params, x, [r], v=v, fg=fg)
    start = s.owner().copy()
    _follow(gs, ref, s, 90, 5)
    assert (s.owner() != start).sum() >= 5
    saved = gs.state_save()
    gs.step(40)
    gs.state_load(saved)
    _follow(gs, ref, s, 120, 5)
    for one in (gs, ref, s):
        one.close()


@pytest.mark.parametrize("fixed", [0, 1])
def test_small_sphere_hits_a_large_one(fixed):
    """It runs 1.2 nodes deep into the large one, nodes change hands, and it leaves again."""
    x, r = np.array([[15.3, 15.2, 15.9], [32.1, 15.6, 16.2]]), np.array([13.0, 3.0])
    v = np.array([[0.0, 0.0, 0.0], [-0.06, 0.0, 0.0]])
    params = dict(nx=44, ny=31, nz=32, tau=0.8, rho_f=1.0, bc=(0,) * 6, rho_p=30.0, E=5.0, nu=0.2, max_particles=2,
                  max_radius=13.0, rest_free=True, node_lists=0)
    gs, ref, s = _pair(params, x, r, v=v, fixed=np.array([fixed, 0], np.uint8))
    _follow(gs, ref, s, 60, 2)
    p = gs.particles_get(0)["x"]
    assert np.linalg.norm(p[0] - p[1]) < 15.0
    _follow(gs, ref, s, 100, 2)
    p = gs.particles_get(0)["x"]
    assert np.linalg.norm(p[0] - p[1]) > 17.0
    for one in (gs, ref, s):
        one.close()


def test_reprojection_of_one_large_sphere_at_rest():
    """Radius 60 at rest: the re-projection takes less than a third of the fluid kernel's time."""
    from paper_1808_08921_amd.lbdem import LatticeSet

    params = dict(nx=160, ny=160, nz=160, tau=0.8, rho_f=1.0, bc=(0,) * 6, rho_p=5000.0, max_particles=1,
                  max_radius=60.0)
    with LatticeSet([params], precision="fp32") as gs:
        gs.particles_set(0, [[80.31, 79.83, 80.17]], [60.0], fixed=[1])
        gs.step(20)
        gs.timing_enable()
        gs.step(20)
        _, _, fluid, remap, _ = gs.timing_read()[0]
    assert remap < fluid / 3.0
