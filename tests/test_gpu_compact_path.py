"""Compact storage beside node lists that keep solid nodes' slots: the 16-bit storages' path
by ranks (source rows with one and several 64-node words, the last one ragged, periodic faces
whose neighbour is in the row's other end, a sphere across a face, waves that hold nodes at a
wall or a density face and so take the general path).  Node lists take the general path at
every node and perform the same arithmetic, so populations agree bit for bit."""
import numpy as np
import pytest

from paper_1808_08921_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("shape,bc,y", [((33, 9, 7), (0,) * 6, 0.4), ((64, 8, 9), (0, 0, 0, 0, 2, 2), 4.0),
                                        ((70, 17, 12), (1, 1, 0, 0, 1, 1), 16.6), ((130, 7, 8), (0, 0, 1, 1, 0, 0), 3.4),
                                        ((8, 12, 70), (0,) * 6, 5.0)])
def test_compact_storage_matches_node_lists(precision, shape, bc, y):
    from paper_1808_08921_amd.lbdem import LatticeSet

    nx, ny, nz = shape
    f0 = inputs.random_populations(shape, seed=11)
    x = np.array([[0.3 if bc[0] == 0 else nx / 2.0, y, nz / 2.0 - 0.2]])
    r = np.array([2.1])
    params = dict(nx=nx, ny=ny, nz=nz, tau=0.8, rho_f=1.0, bc=bc, probe_z=(0, nz - 1), rho_p=2.0, max_radius=2.5,
                  max_particles=1, wave=inputs.WAVE_SINE, amp=1e-3, omega=0.3, t_n=100)
    got = []
    for node_lists in (1, 2):
        with LatticeSet([params], precision=precision, node_lists=node_lists, graph_steps=4) as gs:
            gs.particles_set(0, x, r, fixed=[1])
            gs.set_populations(0, f0)
            gs.step(13)
            gs.check()
            got.append((gs.owner(0), gs.populations(0)))
    own = got[0][0]
    assert np.array_equal(got[1][0], own) and (own >= 0).any()
    assert np.array_equal(got[0][1][:, own < 0], got[1][1][:, own < 0])


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shape", [(33, 41, 20), (32, 32, 18), (65, 31, 16), (30, 20, 24)])
def test_moving_sphere_rebuilds_compact_planes(precision, shape):
    """Lists rebuilt under a sphere that crosses the whole lattice, in planes of more than, of
    exactly, of twice less one and of less than the 1024 cells a workgroup scans at a time:
    nodes behind the first change of a plane's list change slots and keep their values."""
    from paper_1808_08921_amd.lbdem import LatticeSet

    nx, ny, nz = shape
    f0 = inputs.random_populations(shape, seed=12)
    params = dict(nx=nx, ny=ny, nz=nz, tau=0.8, rho_f=1.0, bc=(0,) * 6, rho_p=1e4, max_radius=4.5, max_particles=1)
    got = []
    for node_lists in (1, 2):
        with LatticeSet([params], precision=precision, node_lists=node_lists, graph_steps=4) as gs:
            gs.particles_set(0, np.array([[4.3, ny / 2 - 0.4, nz - 1.8]]), np.array([4.1]), v=np.array([[0.08, 0.03, 0.05]]))
            gs.set_populations(0, f0)
            gs.step(240)
            gs.check()
            got.append((gs.owner(0), gs.populations(0)))
    own = got[0][0]
    assert np.array_equal(got[1][0], own) and (own >= 0).any()
    assert np.array_equal(got[0][1][:, own < 0], got[1][1][:, own < 0])
