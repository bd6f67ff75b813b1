"""The space stage where a row is split over workgroups (few frequencies, long rows), with its own
kernel for the ridge, and where rows share a workgroup: sizes on both sides of each rule.
Reference and tolerance as for the other sizes: the sums as written, phases in extended
precision, and sum |x| times the unit roundoff times the largest phase's and the sums' share.
And few frequencies are not slower than many: one row of the spectrum on one compute unit took
as long as a row on every one of them."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.mark.parametrize("nt,nz,nw,nk", [
    (9, 33, 2, 3972), (9, 33, 2, 3971),        # either side of 131072 elements a row
    (5, 600, 3, 256), (5, 600, 3, 257),        # one part, and one column in a second
    (3, 8, 5, 16385), (3, 7, 5, 18800),        # few columns: split from eight on
    (4, 40, 511, 3300), (4, 40, 512, 3300),    # split, four rows and two; not split
    (3, 31, 40, 4300), (3, 32, 40, 4300),      # loads of four and of eight columns in flight
    (3, 7, 512, 257), (3, 7, 513, 256), (3, 5, 1024, 1000), (3, 5, 1025, 1024),
])
def test_rows_of_the_space_stage(nt, nz, nw, nk):
    import torch

    from paper_1808_08921_amd import lbdem

    rng = np.random.default_rng(nt + nz + nk)
    x = rng.standard_normal((nt, nz))
    zpos = np.sort(rng.uniform(0.0, 50.0, nz))
    t0, w0, dw, k0, dk = 3.0, 0.02, 0.9 / nw, -0.4, 0.8 / nk
    F, ridge = lbdem.st_dft(torch.tensor(x, device="cuda"), zpos, t0, w0, dw, nw, k0, dk, nk)
    alone = lbdem.st_dft(torch.tensor(x, device="cuda"), zpos, t0, w0, dw, nw, k0, dk, nk, ridge=False)
    assert torch.equal(F, alone)
    F, ridge = F.cpu().numpy(), ridge.cpu().numpy()
    w, k = w0 + np.arange(nw) * dw, k0 + np.arange(nk) * dk
    ph = np.longdouble(w)[:, None] * (np.longdouble(t0) + np.arange(nt))[None, :]
    G = (np.cos(ph).astype(float) - 1j * np.sin(ph).astype(float)) @ x
    pk = np.longdouble(zpos)[:, None] * np.longdouble(k)[None, :]
    want = G @ (np.cos(pk).astype(float) + 1j * np.sin(pk).astype(float))
    phase = np.abs(w).max() * (t0 + nt) + np.abs(k).max() * 50.0
    assert np.abs(F - want).max() <= np.abs(x).sum() * EPS * (4.0 * phase + 256.0 + nt + nz)
    p = F.real * F.real + F.imag * F.imag
    top = p.max(axis=1)
    assert np.all((ridge >= 0) & (ridge < nk))
    assert np.all(p[np.arange(nw), ridge] >= top * (1.0 - 4.0 * EPS))


def test_ridge_of_split_rows_with_ties_and_nothing():
    import torch

    from paper_1808_08921_amd import lbdem

    for value, want in ((0.0, 0), (float("nan"), -1)):
        x = torch.full((7, 40), value, dtype=torch.float64, device="cuda")
        _, ridge = lbdem.st_dft(x, np.arange(40.0), 0.0, 0.1, 0.01, 9, 0.0, 0.01, 5000)
        assert (ridge.cpu().numpy() == want).all()


def test_one_frequency_is_not_slower_than_a_hundred():
    """One row of 4096 wavenumbers from 4096 columns is a hundredth of the work of a hundred rows."""
    import torch

    from paper_1808_08921_amd import lbdem

    nt, nz, nk = 64, 4096, 4096
    x = torch.randn((nt, nz), dtype=torch.float64, device="cuda")
    z = torch.arange(nz, dtype=torch.float64, device="cuda")

    def best(nw):
        took = []
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            lbdem.st_dft(x, z, 0.0, 0.1, 0.01, nw, 0.0, 0.001, nk)
            torch.cuda.synchronize()
            took.append(time.perf_counter() - t)
        return min(took)

    assert best(1) < 0.8 * best(100)
