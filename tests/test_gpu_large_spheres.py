"""Sets of few large spheres: the link pass cuts the planes around a sphere into more slabs, from
a radius of 15 on, as the room of the set says (max_radius), up to 64.  State against the oracle
on both sides of each rule; and the time of the link pass beside the fluid kernel's, which does
not grow with the radius as the eight waves of one workgroup would."""
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
