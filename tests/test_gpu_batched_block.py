"""The block form of the FP32 cycle and the zero-start sweeps in batches.

Box sizes of every tile and tail of the form as finest and coarse levels (16, 24, 32, 48, 64) and
above it (96, 128, 192), one box of each, with one and two inner cycles (the second from a non-zero
start), against the FP64 solve of each box alone. Tolerance: as in test_gpu_block_cycle, relative
residuals of 1e-10 leave at most 2e-10 (0.5 n / 2 pi)^2.
"""
import math

import numpy as np
import pytest

import inputs
from gpu_util import announce, dev, host, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402

SIZES = [16, 24, 32, 48, 64, 96, 128, 192]


@pytest.mark.parametrize("inner", [1, 2])
def test_batch_of_every_tile(inner):
    require_gpu()
    announce(f"batched block cycle, {inner} inner cycles")
    deltas = [dev(inputs.lognormal(n, 0.6, 2.5, 40 + n)) for n in SIZES]
    with mr.Batch(SIZES, tol=1e-10, inner_cycles=inner) as b:
        thetas, infos = b.solve(deltas, check=False)
    for n, delta, theta, info in zip(SIZES, deltas, thetas, infos):
        assert info.rel_residual <= 1e-10, (n, info)
        with mr.Context(n, tol=1e-10) as c:
            ref = host(c.solve(delta)[0])
        bound = 2e-10 * max(1.0, (0.5 * n / (2.0 * math.pi)) ** 2)
        assert np.linalg.norm(host(theta) - ref) <= bound * np.linalg.norm(ref), n
