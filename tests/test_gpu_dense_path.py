"""The dense tiles' fixed-offset path beside the general one: odd extents on both sides of a
tile, periodic faces (the offsets wrap), walls and density faces (general path), a sphere in
between (waves of both kinds in a workgroup), every storage, with and without particles (a
set without runs no link, motion and refresh kernels).  Node lists take the general path at
every node and perform the same arithmetic, so both mappings agree bit for bit; FP64 agrees
with the oracle to the rounding of 12 steps (1e-13 on populations of order one)."""
import numpy as np
import pytest

import oracle
from paper_1808_08921_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("sphere", [False, True])
@pytest.mark.parametrize("shape,bc", [((33, 9, 7), (0,) * 6), ((70, 17, 12), (0, 0, 0, 0, 2, 2)),
                                      ((13, 11, 10), (1, 1, 0, 0, 1, 1)), ((8, 8, 2), (0, 0, 0, 0, 0, 0))])
def test_dense_tiles_match_node_lists(precision, sphere, shape, bc):
    from paper_1808_08921_amd.lbdem import LatticeSet

    nx, ny, nz = shape
    if sphere and min(shape) < 7:
        pytest.skip("no room for a sphere")
    f0 = inputs.random_populations(shape, seed=9)
    wave = dict(wave=inputs.WAVE_SINE, amp=1e-3, omega=0.3, t_n=100)
    x, r = np.array([[nx / 2 + 0.3, ny / 2 - 0.2, nz / 2]]), np.array([2.1])
    params = dict(nx=nx, ny=ny, nz=nz, tau=0.8, rho_f=1.0, bc=bc, probe_z=(0, nz - 1), rho_p=2.0, max_radius=2.5,
                  max_particles=1 if sphere else 0, **wave)
    got = []
    for node_lists in (0, 1):
        with LatticeSet([params], precision=precision, node_lists=node_lists, graph_steps=4) as gs:
            if sphere:
                gs.particles_set(0, x, r, fixed=[1])
            gs.set_populations(0, f0)
            gs.step(13)
            gs.check()
            got.append((gs.owner(0), gs.populations(0)))
    own = got[0][0]
    assert np.array_equal(got[1][0], own)
    assert np.array_equal(got[0][1][:, own < 0], got[1][1][:, own < 0])
    if precision != "fp64":
        return
    s = oracle.Sim(nx, ny, nz, tau=0.8, bc=bc, probe_z=(0, nz - 1), rho_p=2.0, **wave)
    if sphere:
        s.set_particles(x, r, fixed=[1])
    s.set_populations(f0)
    s.step(13)
    assert np.array_equal(own, s.owner())
    assert np.abs(s.populations() - got[0][1])[:, own < 0].max() <= 1e-13
    s.close()
