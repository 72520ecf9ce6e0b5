"""Coarse work enqueued before a cycle's residual norm is known (meshes whose finest level runs in the block
form): a solve that stops right after such work leaves nothing behind.

A tolerance that the first cycle meets stops with the coarse part enqueued for nothing; a limit of one or
two cycles and the ordinary tolerance stop without. Each is compared bit for bit with the same call on a new
context, in an order that mixes them, and so is a call on the same context afterwards: launches, sums and
their orders are the same ones.
"""
import numpy as np
import pytest
import torch

import inputs
from gpu_util import announce, dev, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402


@pytest.mark.parametrize("n", [16, 40, 80])
def test_stopping_after_work_enqueued_ahead(n):
    require_gpu()
    announce(f"run ahead n={n}")
    delta = dev(inputs.lognormal(n, 0.7, 2.5, 40 + n))
    g = dev(np.random.default_rng(n).standard_normal((n, n, n)))

    def calls(c, tol, max_cycles):
        c.set_opts(tol=tol, max_cycles=max_cycles)
        theta, info = c.solve(delta, check=False)
        grad, ginfo = c.adjoint_solve(delta, theta, g, check=False)
        return theta, grad, info.cycles, ginfo.cycles

    cases = [(0.9, 100), (1e-10, 1), (1e-10, 100), (1e-3, 100), (1e-10, 2), (1e-10, 100)]
    with mr.Context(n) as one:
        for tol, limit in cases:
            got = calls(one, tol, limit)
            with mr.Context(n) as fresh:
                want = calls(fresh, tol, limit)
            assert got[2:] == want[2:]
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
