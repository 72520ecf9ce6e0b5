"""The 48- and 40-column tiles of the pipelined sweeps (sweep.hip, mixed.hip).

Sizes: one tile across a row of columns (96, 80) and two (192, 160); the smallest chunks of planes and
one chunk of all. Sweeps are compared with the oracle's element by element: FP64 to 1e-12 of the
field's scale (rounding order only), FP32 with the states and the tolerance of the other FP32 schedules. The
launches whose tile is chosen by timing (defect, right-hand side, residual, operator product) are reached
through solves, FP64 and mixed, against a context whose finest sweeps run a narrow tile: each solve to 1e-11, which leaves errors of at most
1e-11 (0.5 n / 2 pi)^2 < 2.4e-9 at 192^3 in theta each; 5e-9 between them.
"""
import numpy as np
import pytest

import inputs
from gpu_util import announce, dev, host, require_gpu
from oracle import multigrid as omg
from test_gpu_linear import TOL32, _lin_sweep_ref
from test_gpu_linear import _state as _lin_state
from test_gpu_schedules import C_SHIFT

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402

TILES = [(96, 48), (192, 48), (80, 40), (160, 40)]


def _state(n, seed):
    delta = inputs.lognormal(n, 0.8, 2.0, seed)
    theta = inputs.grf(n, 1.5, seed + 1)
    theta *= 0.3 / theta.std()
    return delta, theta


@pytest.mark.parametrize("n,tm", TILES)
def test_fp64_sweeps_match_oracle(n, tm):
    require_gpu()
    delta, theta = _state(n, 300 + n)
    ref = omg.rb_sweep(theta, delta, None, 1.0, m=C_SHIFT)
    scale = np.abs(ref).max()
    d_delta, d_theta = dev(delta), dev(theta)
    with mr.Context(n) as c:
        for tj in (8, 16):
            for nch in (n // 16, n // 8, 1):
                sched = (mr.MR_SCHED_PIPELINED, tm, tj, nch)
                announce(f"wide tile {sched} n={n}")
                c.set_schedule(0, sched)
                out, _ = c.sweep(d_delta, d_theta, cshift=C_SHIFT)
                err = np.max(np.abs(host(out) - ref))
                assert err <= 1e-12 * scale, f"{sched}: max abs diff {err:.3e}"


@pytest.mark.parametrize("n,tm", TILES[::2])
def test_fp32_sweeps_match_oracle(n, tm):
    require_gpu()
    delta, theta, e, rhs = _lin_state(n, 400 + n)
    ref = _lin_sweep_ref(theta, delta, e, 1.0, rhs, C_SHIFT)
    scale = np.abs(ref).max()
    with mr.Context(n, precision=mr.PREC_MIXED) as c:
        for kind in (mr.MR_SCHED_PIPELINED, mr.MR_SCHED_TILED):
            for tj in (8, 16):
                sched = (kind, tm, tj, n // 16)
                announce(f"wide FP32 tile {sched} n={n}")
                got = host(c.lin_sweep(dev(delta), dev(theta), dev(e), rhs=dev(rhs), cshift=C_SHIFT, sched=sched))
                err = np.max(np.abs(got - ref))
                assert err <= TOL32 * scale, f"{sched}: max abs diff {err:.3e} (scale {scale:.3e})"


@pytest.mark.parametrize("n,tm", TILES)
def test_solves_match_the_narrow_tile(n, tm):
    require_gpu()
    announce(f"wide tile solves n={n}")
    delta = inputs.lognormal(n, 0.8, 2.5, 500 + n)
    d = dev(delta)
    out = []
    narrow = (mr.MR_SCHED_PIPELINED, 16, 16, n // 16) if tm == 48 else (mr.MR_SCHED_TILED, 8, 16, 8)
    for sched in ((mr.MR_SCHED_PIPELINED, tm, 8, n // 16), narrow):
        with mr.Context(n, tol=1e-11) as c:
            c.set_schedule(0, sched)
            theta, info = c.solve(d)
            assert info.status == 0
            out.append(host(theta))
    with mr.Context(n, tol=1e-11, precision=mr.PREC_MIXED) as c:
        theta, info = c.solve(d)
        assert info.status == 0
        out.append(host(theta))
    for other in out[1:]:
        assert np.linalg.norm(out[0] - other) <= 5e-9 * np.linalg.norm(other)
