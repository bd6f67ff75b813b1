"""Sets with room for exactly 256 particles, whose link kernel moves them, and for exactly one
more, which have the motion kernel: bit for bit the same, and neither raises an error (but for
the particle over the speed limit)."""
import numpy as np
import pytest

from test_gpu_motion_fused import _run

pytestmark = pytest.mark.gpu

ERRORS = 0x2 | 0x8 | 0x10 | 0x40 | 0x80 | 0x100 | 0x400


@pytest.mark.parametrize("precision", ["fp64", "fp16"])
@pytest.mark.parametrize("n", [1, 7, 60, 256])
def test_both_sides_of_256_places(precision, n):
    rng = np.random.default_rng(n)
    side = int(np.ceil(n ** (1 / 3)))
    cell = 5.2  # (no node borders more than four spheres)
    grid = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    shape = (max(10, int(np.ceil(side * cell))),) * 3
    x = 0.5 * cell + cell * grid + rng.uniform(-0.2, 0.2, (n, 3))
    r = rng.uniform(2.1, 2.5, n)
    v = rng.uniform(-0.05, 0.05, (n, 3))
    fixed = (np.arange(n) % 5 == 4).astype(np.uint8)
    if n == 7:
        v[0] = (0.4, 0.0, 0.0)
    a = _run(precision, shape, x, r, v, fixed, 256 - n)
    b = _run(precision, shape, x, r, v, fixed, 257 - n)
    assert a[0] & ERRORS == (0x10 if n == 7 else 0) and a[0] == b[0]
    assert np.array_equal(a[1], b[1])
    fluid = a[1] < 0
    assert np.array_equal(a[2][:, fluid], b[2][:, fluid])
    for k in a[3]:
        assert np.array_equal(a[3][k], b[3][k]), k
