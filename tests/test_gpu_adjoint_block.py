"""The block form of the adjoint cycle on meshes of 80^3 cells and below (adj_block.hip).

Every compiled tile as the finest level (20, 24: 4^3; 32; 40; 48; 64, 80) and below the plain half-sweeps (96,
160), with the three tails (8^3 over 4^3, 12^3 over 6^3, 10^3), against the same solve with the row
kernels on every level (MR_FLAG_ADJ_ROWS). Tolerance: each gradient solves its system to a relative
residual of 1e-10, which leaves an error of at most that times the ratio of the mean square wavenumber
to the smallest one, (0.5 n / 2 pi)^2.
"""
import math

import numpy as np
import pytest

import inputs
from gpu_util import announce, dev, host, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402


@pytest.mark.parametrize("n,depth", [(20, 0), (24, 0), (32, 2), (40, 0), (48, 0), (64, 0), (80, 0), (96, 0), (160, 0)])
def test_block_form_matches_row_kernels(n, depth):
    require_gpu()
    announce(f"adjoint block cycle n={n} depth={depth}")
    delta = dev(inputs.lognormal(n, 0.7, 2.5, 90 + n))
    g = dev(np.random.default_rng(n).standard_normal((n, n, n)))
    with mr.Context(n, tol=1e-12) as c:
        theta, _ = c.solve(delta)
    grads, cycles = [], []
    for flags in (0, mr.MR_FLAG_ADJ_ROWS):
        with mr.Context(n, tol=1e-10, flags=flags) as c:
            out, info = c.adjoint_solve(delta, theta, g, anderson_depth=depth)
        grads.append(host(out))
        cycles.append(info.cycles)
    print(f"n={n}: cycles {cycles}")
    assert abs(cycles[0] - cycles[1]) <= 1
    bound = 2e-10 * max(1.0, (0.5 * n / (2.0 * math.pi)) ** 2)
    assert np.linalg.norm(grads[0] - grads[1]) <= bound * np.linalg.norm(grads[1])
