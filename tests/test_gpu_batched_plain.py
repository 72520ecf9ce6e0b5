"""Batches whose coarse levels run the plain launches: any number of sweeps but two before and two after.

The zero-start sweeps on every level, the cleared coarse meshes (before the coarsest sweeps, and on every
level when there is no sweep before the restriction) and the one-workgroup coarsest mesh, on boxes of 4 2^k and 6 2^k
cells a side from the smallest to one above the block form's limits, with one and two inner cycles, against
the FP64 solve of each box alone. Tolerance: as in test_gpu_batched_block, times 4 because on the smallest
meshes the field has few modes besides the longest and the Jacobian's coefficients, down to about a
quarter of the Laplacian's in single cells, are not averaged out. Sizes that batches have no tiles for
(10 2^k, whose hierarchy holds a 20^3 mesh) are refused before any work on the boxes.
"""
import math

import numpy as np
import pytest

import inputs
from gpu_util import announce, dev, host, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402

SIZES = [8, 12, 16, 24, 32, 48, 64, 96, 128]


@pytest.mark.parametrize("inner", [1, 2])
@pytest.mark.parametrize("npre,npost", [(1, 1), (0, 2), (3, 2)])
def test_plain_coarse_levels(npre, npost, inner):
    require_gpu()
    announce(f"batched plain launches, sweeps {npre}/{npost}, {inner} inner cycles")
    deltas = [dev(inputs.lognormal(n, 0.6, 2.5, 40 + n)) for n in SIZES]
    with mr.Batch(SIZES, tol=1e-10, npre=npre, npost=npost, inner_cycles=inner) as b:
        for _ in range(2):   # the second replays the same graph on buffers that are no longer zero
            thetas, infos = b.solve(deltas, check=False)
    for n, delta, theta, info in zip(SIZES, deltas, thetas, infos):
        assert info.rel_residual <= 1e-10, (n, info)
        with mr.Context(n, tol=1e-10) as c:
            ref = host(c.solve(delta)[0])
        bound = 8e-10 * max(1.0, (0.5 * n / (2.0 * math.pi)) ** 2)
        assert np.linalg.norm(host(theta) - ref) <= bound * np.linalg.norm(ref), n


@pytest.mark.parametrize("n", [20, 40, 80, 160])
def test_sizes_without_tiles_are_refused(n):
    require_gpu()
    announce(f"batched size {n} refused")
    with pytest.raises(mr.MRError):
        mr.Batch([16, n])
