"""Link entries found from the sphere's equation, and re-projection candidates found the same
way, at the sizes where their slabs, runs and queues can go wrong: a sphere smaller than a
node distance, one whose slabs hold more candidates than the LDS list, one that crosses
periodic faces on every axis, planes cut by walls, and a fast one whose reference point moves
every other step.  Node maps exact and particles within 1e-10 of the oracle, the bars of the
other parity tests."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CASES = {
    # shape, faces, centre, radius, velocity, steps
    "radius below a node distance": ((9, 9, 9), (0,) * 6, (4.3, 4.6, 4.1), 0.4, (0.05, 0.02, -0.03), 20),
    "a slab of many candidates": ((70, 70, 70), (0,) * 6, (34.7, 35.2, 33.9), 27.3, (0.02, -0.01, 0.03), 6),
    "across every periodic face": ((21, 23, 19), (0,) * 6, (0.2, 22.7, 0.1), 6.3, (-0.1, 0.12, -0.08), 24),
    "cut by walls": ((20, 18, 22), (1,) * 6, (3.1, 14.6, 2.2), 5.7, (0.04, -0.05, 0.06), 24),
    "a reference point that moves": ((26, 24, 40), (0, 0, 0, 0, 1, 1), (12.4, 11.8, 9.3), 5.2, (0.1, 0.1, 0.2), 40),
}


@pytest.mark.parametrize("node_lists", [0, 2])
@pytest.mark.parametrize("name", sorted(CASES))
def test_moving_sphere_matches_oracle(name, node_lists):
    from paper_1808_08921_amd.lbdem import LatticeSet

    (nx, ny, nz), bc, x, r, v, steps = CASES[name]
    x, v, w = np.array([x]), np.array([v]), np.array([[2e-3, -1e-3, 3e-3]])
    params = dict(nx=nx, ny=ny, nz=nz, tau=0.9, rho_f=1.0, bc=bc, E=10.0, nu=0.2, mu=0.0, rho_p=3.0, probe_z=(0, nz // 2),
                  max_particles=1, max_radius=r + 0.2)
    s = oracle.Sim(nx, ny, nz, tau=0.9, bc=bc, E=10.0, nu=0.2, mu=0.0, rho_p=3.0, probe_z=(0, nz // 2))
    s.set_particles(x, [r], v=v, w=w)
    s.step(steps)
    o = s.particles()
    with LatticeSet([params], precision="fp64", node_lists=node_lists, graph_steps=4) as gs:
        gs.particles_set(0, x, [r], v=v, w=w)
        gs.step(steps)
        g = gs.particles_get(0)
        own = gs.owner(0)
        gs.check()
    assert np.array_equal(own, s.owner())
    for k in ("x", "v", "w", "force", "torque"):
        scale = np.abs(o[k]).max() if k != "torque" else max(np.abs(o[k]).max(), np.abs(o["force"]).max())
        assert np.abs(g[k] - o[k]).max() <= 1e-10 * scale, k
    s.close()
