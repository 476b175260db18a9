"""Reciprocals of the Sinkhorn-Knopp half steps where a line's sum leaves the normal range (below 2^-126 = e^-87.3): H_res
against the oracle, for each count of lanes per token and one token per lane; and the division's bits where sums are near 1."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_05732_amd as mhcl
from gpu_harness import rel_err, to_np64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,T", [(2, 40), (4, 40), (4, 16384), (3, 90000), (5, 40), (5, 40000)])
@pytest.mark.parametrize("low", [-60.0, -86.5, -87.5, -88.0, -89.0])
def test_sums_below_the_normal_range(n, T, low):
    C = 64
    d = mhcl.Desc(n, C, T, mhcl.BF16, mhcl.RES_SK)
    z = np.zeros((n, n), dtype=np.float32)
    z[:, 1] = low - 0.1 * np.arange(n)                      # the whole column small
    b = torch.cat([torch.from_numpy(z).flatten(), torch.zeros(2 * n)]).cuda()
    x, W = torch.ones(T, n, C, device="cuda", dtype=torch.bfloat16), torch.zeros(n * C, n * n + 2 * n, device="cuda")
    e = lambda *s: torch.empty(s, device="cuda")  # noqa: E731
    H = e(T, n, n)
    mhcl.mhcl_coeffs(d, x, W, b, torch.ones(3, device="cuda"), H, e(T, n), e(T, n), mhcl.binding.new_workspace(d, mhcl.OP_COEFFS))
    ref = oracle.coeffs_sk(to_np64(x[:1]), to_np64(W), to_np64(b), np.ones(3))[0]
    # the entries of that column are fp32 subnormals of e^-89.4 at the least: 2^-149 of them is 1e-6, of which a
    # quotient keeps up to n; fp32 sums and products over 40 half steps add less
    assert rel_err(to_np64(H[:1]), ref) <= 1e-5
    assert torch.equal(H, H[:1].expand_as(H))


@pytest.mark.parametrize("n", [2, 4])
@pytest.mark.parametrize("T", [8000, 40000])          # an entry per lane, a row per lane
def test_a_step_has_the_bits_of_one_with_the_division(n, T):
    C, f = 64, np.float32
    gen = torch.Generator(device="cuda").manual_seed(n)
    normal = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)  # noqa: E731
    x, W, b = normal(T, n, C).to(torch.bfloat16), normal(n * C, n * n + 2 * n) * 0.1, normal(n * n + 2 * n)
    e = lambda *s: torch.empty(s, device="cuda")  # noqa: E731

    def after(steps):
        d, H = mhcl.Desc(n, C, T, mhcl.BF16, mhcl.RES_SK, sk_iters=steps), e(T, n, n)
        mhcl.mhcl_coeffs(d, x, W, b, torch.ones(3, device="cuda"), H, e(T, n), e(T, n), mhcl.binding.new_workspace(d, mhcl.OP_COEFFS))
        return H.cpu().numpy()

    def pairs(v, axis):                               # the order of both sums over four is one of pairs
        a, b = np.split(v, 2, axis) if axis == 1 else (v[:, :, 0::2], v[:, :, 1::2])
        s = a + b
        return s if n == 2 else s.take([0], axis) + s.take([1], axis)

    ties = 0
    for steps in (1, 3, 19):
        H, want = after(steps), after(steps + 1)
        col = pairs(H, 1)
        H = H * (f(1) / col)
        row = pairs(H, 2)
        H = H * (f(1) / row)
        assert H.dtype == f and np.array_equal(H, want), steps
        ties += int((col == f(1) - f(2) ** -24).sum() + (row == f(1) - f(2) ** -24).sum())
    assert ties > 100                                 # sums one step below 1, whose reciprocals lie next to a tie, are among them
