"""The gather from theta in pairs along z against the gather from the mesh field, bit for bit: both form the
same differences and sums in the same order. Particles in every cell of the rows' ends (where single
points across the seam replace half a pair), on the smallest mesh, one with a row longer than a
wavefront, and one of more than 4 GiB, whose offsets need 64 bits.
"""
import numpy as np
import pytest
import torch

from gpu_util import announce, dev, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402


@pytest.mark.parametrize("n", [4, 6, 80, 1024])
def test_pairs_match_the_mesh_field(n):
    require_gpu()
    announce(f"lagrangian rows n={n}")
    rng = np.random.default_rng(n)
    pos = rng.uniform(0.0, n, (20000, 3))
    ends = np.array([0, 1, 2, n - 3, n - 2, n - 1])
    pos[:9000] = ends[rng.integers(0, 6, (9000, 3))] + rng.uniform(0.0, 1.0, (9000, 3))
    gen = torch.Generator(device="cuda").manual_seed(n)
    theta = torch.randn((n, n, n), dtype=torch.float64, device="cuda", generator=gen)
    with mr.Context(n) as c:
        announce(f"lagrangian rows n={n}: context")
        a, _ = c.lagrangian(theta, dev(pos))
        b, psi = c.lagrangian(theta, dev(pos), want_psi=True)
    del psi
    assert torch.equal(a, b)
