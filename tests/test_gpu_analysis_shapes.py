"""The folded time stage, the row-blocked space stage with its ridge and the scanned fit at the
edges of their tiles: records of one row up to several segments with odd lengths, one column up
to several tiles, frequencies and wavenumbers around the tile sizes, more columns than a wave or
the LDS copy holds.  Reference: the sums as written, phases in extended precision.  Tolerance of
F: sum |x| times the unit roundoff times (four times the largest phase, for the rounded products
omega t and kappa z; 256, for 64 rotations between exact phases; one per term added in a
row)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.mark.parametrize("nt,nz,nw,nk", [(1, 1, 1, 1), (2, 3, 31, 65), (7, 16, 32, 64), (63, 17, 33, 300),
                                         (64, 8, 64, 63), (65, 33, 5, 1025), (257, 24, 130, 100), (1000, 2, 513, 7),
                                         (2500, 5, 1030, 130), (4097, 65, 40, 33)])
def test_spectrum_at_tile_edges(nt, nz, nw, nk):
    import torch

    from paper_1808_08921_amd import lbdem

    rng = np.random.default_rng(nt + nz)
    x = rng.standard_normal((nt, nz))
    zpos = np.sort(rng.uniform(0.0, 50.0, nz))
    t0, w0, dw, k0, dk = 3.0, 0.02, 0.9 / nw, -0.4, 0.8 / nk
    F, ridge = lbdem.st_dft(torch.tensor(x, device="cuda"), zpos, t0, w0, dw, nw, k0, dk, nk)
    F, ridge = F.cpu().numpy(), ridge.cpu().numpy()
    w, k = w0 + np.arange(nw) * dw, k0 + np.arange(nk) * dk
    ph = np.longdouble(w)[:, None] * (np.longdouble(t0) + np.arange(nt))[None, :]
    G = (np.cos(ph).astype(float) - 1j * np.sin(ph).astype(float)) @ x
    pk = np.longdouble(zpos)[:, None] * np.longdouble(k)[None, :]
    want = G @ (np.cos(pk).astype(float) + 1j * np.sin(pk).astype(float))
    phase = np.abs(w).max() * (t0 + nt) + np.abs(k).max() * 50.0
    tol = np.abs(x).sum() * EPS * (4.0 * phase + 256.0 + nt + nz)
    assert np.abs(F - want).max() <= tol
    p = F.real * F.real + F.imag * F.imag
    top = p.max(axis=1)
    assert np.all((ridge >= 0) & (ridge < nk))
    # (the device may fuse the two products' sum: a relative roundoff)
    assert np.all(p[np.arange(nw), ridge] >= top * (1.0 - 4.0 * EPS))


def test_ridge_of_ties_and_of_nothing():
    import torch

    from paper_1808_08921_amd import lbdem

    for value, want in ((0.0, 0), (float("nan"), -1)):
        x = torch.full((70, 4), value, dtype=torch.float64, device="cuda")
        _, ridge = lbdem.st_dft(x, np.arange(4.0), 0.0, 0.1, 0.01, 9, 0.0, 0.01, 200)
        assert (ridge.cpu().numpy() == want).all()


@pytest.mark.parametrize("nz", [2, 24, 64, 65, 130, 2100])
def test_fit_unwraps_across_waves(nz):
    """A damped wave with columns of zeros (first, in the middle, a whole wave's worth): the fit
    gives back amplitude, damping and wavenumber.  log |P| and the phase carry the record's
    rounding (below 1e-11 at 4000 rows of a stationary wave over whole periods), the slopes
    that over a column spacing of at least one: 1e-9 with room for 2100 sums."""
    import torch

    from paper_1808_08921_amd import lbdem

    nt, om, t0 = 4000, 2.0 * np.pi / 80.0, 5.0
    z = 1.5 * np.arange(nz)
    amp, alpha, k = 0.7 * np.exp(0.4j), 1.0 / (1.5 * nz), 0.5  # (k times the widest gap, 6, below pi)
    t = t0 + np.arange(nt)
    c = amp * np.exp(-(alpha + 1j * k) * z)
    x = np.real(c[None, :] * np.exp(1j * om * t)[:, None])
    out = [] if nz < 24 else [0, 7, 8, 9][: 1 if nz < 65 else 4]
    if nz >= 130:
        out += list(range(64, 67))
    x[:, out] = 0.0
    f = lbdem.wave_fit(torch.tensor(x, device="cuda"), z, t0, om)
    assert f["n_used"] == nz - len(out)
    assert abs(f["A"] - amp) <= 1e-9 and abs(f["alpha"] - alpha) <= 1e-9 and abs(f["k"] - k) <= 1e-9
