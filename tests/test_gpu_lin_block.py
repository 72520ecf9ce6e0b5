"""The block form of the FP32 linear cycle on meshes of 96^3 cells and below (lin_block.h).

Every compiled tile and tail as the finest level of a mixed-precision solve and below the plain sweeps
(128, 160), with the Krylov inner solve (cycles from zero) and with two plain inner cycles (the second
from a non-zero start), against the FP64 solution of the plain launches. Tolerance: as in
test_gpu_block_cycle, relative residuals of 1e-11 leave at most 2e-11 (0.5 n / 2 pi)^2 between the two.
The Krylov inner solve needs no more than two cycles more than with the plain FP32 launches.
"""
import math

import numpy as np
import pytest

import inputs
from gpu_util import announce, dev, host, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402


@pytest.mark.parametrize("n", [20, 24, 32, 40, 48, 64, 80, 96, 128, 160])
def test_block_form_in_the_mixed_solve(n):
    require_gpu()
    announce(f"linear block cycle n={n}")
    delta = dev(inputs.lognormal(n, 0.8, 2.5, 60 + n))
    with mr.Context(n, tol=1e-11, flags=mr.MR_FLAG_TWO_PASS) as c:
        ref = host(c.solve(delta)[0])
    bound = 2e-11 * max(1.0, (0.5 * n / (2.0 * math.pi)) ** 2) * np.linalg.norm(ref)
    cycles = []
    for flags, inner in ((0, 4), (mr.MR_FLAG_TWO_PASS, 4), (mr.MR_FLAG_PLAIN_INNER, 2)):
        with mr.Context(n, tol=1e-11, precision=mr.PREC_MIXED, inner_cycles=inner, flags=flags) as c:
            theta, info = c.solve(delta)
        assert info.status == 0
        assert np.linalg.norm(host(theta) - ref) <= bound
        cycles.append(info.inner_cycles)
    print(f"n={n}: inner cycles {cycles}")
    assert cycles[0] <= cycles[1] + 2
