"""The pass that takes in delta (domain check, colour split, reference norm) and the streaming sums.

At theta = 0 the residual is minus the source's deviation from its mean, 3 (1 + delta)^(1/3) up to a
constant, so every cell of the converted mesh and both reduced sums show in mr_residual. Sizes: strips
of many rows (4, 12), rows that do not divide a strip (96, 160), one strip a row (256) and rows of two
strips with an idle remainder (320). Tolerance: the root is good to a few units in the last place of
values up to about 10, so 1e-13 per cell; the norm ratio is exactly one up to the order of the sums.
"""
import pytest
import torch

from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu

from paper_1709_06350_amd import mr  # noqa: E402


@pytest.mark.parametrize("n", [4, 12, 96, 160, 256, 320])
def test_intake_converts_checks_and_sums(n):
    require_gpu()
    announce(f"intake n={n}")
    g = torch.Generator(device="cuda").manual_seed(n)
    delta = torch.exp(0.5 * torch.randn((n, n, n), generator=g, dtype=torch.float64, device="cuda")) - 1.0
    root = 3.0 * (1.0 + delta).pow(1.0 / 3.0)
    with mr.Context(n) as c:
        r, rel, msum = c.residual(delta, torch.zeros_like(delta))
        assert float((r - (root.mean() - root)).abs().max()) <= 1e-13
        assert abs(rel - 1.0) <= 1e-12 and abs(msum - float(root.mean() - 3.0)) <= 1e-12
        for at, bad in ((0, -1.0), (n ** 3 - 1, float("nan")), (n ** 3 // 2 + 1, float("inf"))):
            worse = delta.clone()
            worse.view(-1)[at] = bad
            with pytest.raises(mr.MRError) as err:
                c.solve(worse)
            assert err.value.code == mr.MR_EDOMAIN
