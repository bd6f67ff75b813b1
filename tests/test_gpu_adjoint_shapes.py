"""The adjoint window's slots (fluid nodes numbered across planes, 64 to a wave) at the sizes
where they can go wrong: planes smaller than a wave, waves that span several probe planes, a
last wave of one node, periodic x with the wrap in another 32-node word, rows of exactly 32
and 33 nodes, a narrow periodic axis, and no particles.  Forward signals within 1e-10 and FP64
gradients within 1e-9 of the oracle's adjoint, the bars of the other adjoint tests."""
import numpy as np
import pytest

import oracle
from paper_1808_08921_amd import inputs

pytestmark = pytest.mark.gpu

STEPS = 17
CASES = {
    # shape, x/y faces, centres, radii
    "planes of 15 nodes": ((3, 5, 40), (0, 0, 1, 1), [], []),
    "one node over a wave": ((5, 1, 13), (1, 1, 0, 0), [], []),
    "rows of 33, periodic x": ((33, 7, 11), (0, 0, 1, 1), [(32.4, 3.1, 5.3)], [2.3]),
    "rows of 32, walls": ((32, 6, 9), (1, 1, 1, 1), [(5.2, 2.9, 4.4), (9.8, 3.0, 4.1)], [2.1, 2.4]),
    "narrow periodic axes": ((8, 8, 14), (0, 0, 0, 0), [(4.1, 3.9, 6.2)], [3.2]),
}


@pytest.mark.parametrize("ckpt", [1, 5, 40])
@pytest.mark.parametrize("name", sorted(CASES))
def test_window_matches_oracle_adjoint(name, ckpt):
    from paper_1808_08921_amd.lbdem import AdjointWindow, LatticeSet

    (nx, ny, nz), side, x, rad = CASES[name]
    x, rad = np.array(x, float).reshape(-1, 3), np.array(rad, float)
    rng = np.random.default_rng(5)
    v, w = 1e-3 * rng.standard_normal(x.shape), 1e-4 * rng.standard_normal(x.shape)
    pz = (1, 2, nz // 2, nz - 1)
    params = dict(nx=nx, ny=ny, nz=nz, tau=0.9, rho_f=1.0, bc=side + (2, 2), wave=inputs.WAVE_SINE, amp=1e-3,
                  omega=2 * np.pi / 12, t_n=50, probe_z=pz, max_particles=len(x), max_radius=3.5)
    target = 1e-4 * rng.standard_normal((STEPS, len(pz)))
    s = oracle.Sim(nx, ny, nz, tau=0.9, bc=side + (2, 2), wave=inputs.WAVE_SINE, amp=1e-3, omega=2 * np.pi / 12, t_n=50,
                   probe_z=pz)
    s.set_particles(x, rad, v=v, w=w)
    s.set_frozen(True)
    P0, *_ = s.adjoint(STEPS, 0.9, 1e-3, np.zeros((STEPS, len(pz))))
    s.close()
    s = oracle.Sim(nx, ny, nz, tau=0.9, bc=side + (2, 2), wave=inputs.WAVE_SINE, amp=1e-3, omega=2 * np.pi / 12, t_n=50,
                   probe_z=pz)
    s.set_particles(x, rad, v=v, w=w)
    s.set_frozen(True)
    _, gt, ga, gv = s.adjoint(STEPS, 0.9, 1e-3, 2.0 * (P0 - target))
    s.close()
    with LatticeSet([params], precision="fp64", graph_steps=0) as gs:
        if len(x):
            gs.particles_set(0, x, rad, v=v, w=w)
        win = AdjointWindow(gs, 0, nsteps=STEPS, ckpt_every=ckpt)
        P = win.forward(0.9, 1e-3, v)
        assert np.abs(P - P0).max() <= 1e-10 * np.abs(P0).max()
        first = win.backward(2.0 * (P - target))
        again = win.backward(2.0 * (P - target))  # the last segment's states recomputed this time
        win.close()
    assert first[0] == again[0] and first[1] == again[1] and np.array_equal(first[2], again[2])
    assert abs(first[0] - gt) <= 1e-9 * abs(gt)
    assert abs(first[1] - ga) <= 1e-9 * abs(ga)
    if len(x):
        assert np.abs(first[2] - gv).max() <= 1e-9 * np.abs(gv).max()
