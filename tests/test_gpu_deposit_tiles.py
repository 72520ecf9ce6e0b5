"""The tile-sorted deposit and its fixed-point weights, bit for bit against integers formed with numpy.

Sizes: tiles 4 points high (32, 96) and 16 (128); one particle, fewer than a chunk of 1024, a chunk and one
more, and more than the 512 chunks of one round. Positions include weights that are ties of the rounding
(multiples of 2^-41), 0 and 1, coordinates on and next to both ends of the box, and some outside. Every
weight product is formed in the same order in doubles and rounded to a multiple of 2^-40 once, and the
integer sums are exact; the final count * scale - 1 may be fused, which moves it by an ulp of the product,
far below one unit of the sums. The TSC weights may be fused as well, by 2^-53, and a contribution next to
a tie then rounds the other way: one unit for each contribution of a cell.
"""
import numpy as np
import pytest

from gpu_util import announce, dev, host, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402


def _axis(x, n, scheme):
    xw = x - n * np.floor(x / n)
    xw = np.where(xw >= n, xw - n, xw)
    xw = np.where(xw < 0.0, 0.0, xw)
    i = np.floor(xw).astype(np.int64)
    f = xw - i
    if scheme == "cic":
        return [i, (i + 1) % n], [1.0 - f, f]
    up = f >= 0.5
    c = (i + up) % n
    d = f - up
    return [(c - 1) % n, c, (c + 1) % n], [0.5 * ((0.5 - d) * (0.5 - d)), 0.75 - d * d, 0.5 * ((0.5 + d) * (0.5 + d))]


def _expected(pos, n, scheme):
    grid, hits = np.zeros(n ** 3, dtype=np.int64), np.zeros(n ** 3, dtype=np.int64)
    (ix, wx), (iy, wy), (iz, wz) = (_axis(pos[:, k], n, scheme) for k in range(3))
    for a in range(len(ix)):
        for b in range(len(iy)):
            for d in range(len(iz)):
                w = np.rint(wx[a] * wy[b] * wz[d] * 2.0 ** 40).astype(np.int64)
                cell = (ix[a] * n + iy[b]) * n + iz[d]
                np.add.at(grid, cell, w)
                np.add.at(hits, cell, 1)
    unit = n ** 3 / (pos.shape[0] * 2.0 ** 40)
    return (grid.astype(float) * unit).reshape(n, n, n), hits.reshape(n, n, n), unit


@pytest.mark.parametrize("scheme", ["cic", "tsc"])
@pytest.mark.parametrize("n,count", [(32, 1), (32, 1023), (96, 1025), (128, 4097), (96, 512 * 1024 + 700)])
def test_sorted_deposit_is_the_integer_sum(scheme, n, count):
    require_gpu()
    announce(f"deposit integers {scheme} n={n} np={count}")
    rng = np.random.default_rng(n + count)
    pos = rng.uniform(0.0, n, (count, 3))
    edge = np.array([0.0, -0.0, 0.5, n - 0.5, np.nextafter(n, 0.0), float(n), -1e-300, 2.0 ** -41, 3 * 2.0 ** -41,
                     1.0 + 2.0 ** -20, n - 2.0 ** -21, -3.25 * n, 7.5 * n, 1e-320])
    k = min(count, 40 * edge.size)
    pos[:k] = edge[rng.integers(0, edge.size, (k, 3))]
    with mr.Context(n) as c:
        got = host(c.deposit(dev(pos), 1.0, scheme))
    rho, hits, unit = _expected(pos, n, scheme)
    bound = 2.0 ** -52 * (rho + 1.0)
    assert bound.max() < 0.5 * unit
    if scheme == "tsc":
        bound = bound + hits * unit
    assert np.all(np.abs(got - (rho - 1.0)) <= bound)
