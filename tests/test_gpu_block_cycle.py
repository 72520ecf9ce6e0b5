"""The block form of the FAS cycle on meshes of 80^3 cells and below (block_cycle.hip).

Sizes: every compiled tile as the finest level (16 and 24: 4^3; 20: 4^3 over a coarsest 10^3; 32:
4 x 4 x 8; 40: 4 x 8 x 8; 48: 8^3; 64 and 80: 8 x 8 x 16) and as a level below the plain sweeps (96, 128, 160).
The reference is the oracle's solution where it is quick, and the library's plain launches
(MR_FLAG_TWO_PASS switches the block form off) elsewhere.

Tolerance: a relative residual of 1e-12 leaves an error in theta of at most that times the ratio of the
field's mean square wavenumber to the smallest one, (0.5 n / 2 pi)^2 < 170 at 160^3: 2e-10 for each
of the two solutions, so 1e-9 between them (the oracle's runs to 1e-11 at n <= 24: factor 4).
"""
import numpy as np
import pytest

import inputs
from gpu_util import announce, dev, host, require_gpu
from oracle import multigrid as omg

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402


def _solve(delta, **opts):
    with mr.Context(delta.shape[0], tol=1e-12, **opts) as c:
        theta, info = c.solve(dev(delta))
    return host(theta), info


@pytest.mark.parametrize("n", [16, 20, 24])
def test_small_meshes_match_oracle(n):
    require_gpu()
    announce(f"block cycle vs oracle n={n}")
    delta = inputs.lognormal(n, 0.7, 2.5, 70 + n)
    theta, info = _solve(delta)
    ref, _ = omg.solve(delta, tol=1e-11)
    assert info.status == 0
    assert np.linalg.norm(theta - ref) <= 1e-9 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [16, 32, 40, 48, 64, 80, 96, 128, 160])
def test_block_form_reaches_the_plain_cycles_solution(n):
    require_gpu()
    announce(f"block cycle vs plain launches n={n}")
    delta = inputs.lognormal(n, 0.9, 2.0, 80 + n)
    theta, info = _solve(delta)
    plain, pinfo = _solve(delta, flags=mr.MR_FLAG_TWO_PASS)
    print(f"n={n}: cycles {info.cycles} (plain {pinfo.cycles})")
    assert abs(info.cycles - pinfo.cycles) <= 1
    assert abs(info.m_shift - pinfo.m_shift) <= 1e-11
    assert np.linalg.norm(theta - plain) <= 1e-9 * np.linalg.norm(plain)


def test_pinned_level_runs_its_own_sweeps():
    require_gpu()
    announce("pinned schedule on a level of the block form")
    delta = inputs.lognormal(64, 0.7, 3.0, 9)
    theta, _ = _solve(delta)
    with mr.Context(64, tol=1e-12) as c:
        c.set_schedule(1, (mr.MR_SCHED_TILED, 16, 16, 4))   # 32^3: the finest level and this one as launches
        pinned, info = c.solve(dev(delta))
    assert info.status == 0
    assert np.linalg.norm(theta - host(pinned)) <= 1e-9 * np.linalg.norm(theta)
