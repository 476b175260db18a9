"""mhcl_post on streams that exceed the 256 MiB last-level cache, where x and y are read past it, and from the sizes on
from which x_out is written past the caches: the bits of the same tokens given in two calls below that size; and the exact
value of a few tokens."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import desc_for, TOL_BF16_OUT, TOL_F32

pytestmark = pytest.mark.gpu


# exactly at the lines of the stores (4 MiB, and 80 MiB with more than 64 logits); one token above and exactly at 256 MiB, rows that divide the cache's size and one that does not
@pytest.mark.parametrize("n,C,T,io", [(4, 1024, 512, "bf16"), (5, 1024, 8192, "bf16"), (4, 4096, 8193, "bf16"), (4, 4096, 8192, "bf16"), (3, 1000, 44740, "bf16"),
                                      (1, 8192, 8193, "f32"), (2, 2056, 16400, "f32")])
def test_large_streams_equal_their_halves(n, C, T, io):
    dt = torch.bfloat16 if io == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(3)
    normal = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    x, y = normal(T, n, C).to(dt), normal(T, C).to(dt)
    H_res, H_post = normal(T, n, n), normal(T, n)

    def post(lo, hi):
        wl = si.Workload("w", n=n, C=C, T=hi - lo, io=io)
        out = torch.full((hi - lo, n, C), float("nan"), device="cuda", dtype=dt)
        mhcl.mhcl_post(desc_for(wl), x[lo:hi], y[lo:hi], H_res[lo:hi], H_post[lo:hi], out)
        return out

    whole, half = post(0, T), T // 8 * 4      # H_post[half:] on a 16-byte boundary
    assert torch.equal(whole, torch.cat([post(0, half), post(half, T)]))
    pick = torch.tensor([0, 1, half, T - 1], device="cuda")
    exact = H_res[pick].double() @ x[pick].double() + H_post[pick].double()[:, :, None] * y[pick].double()[:, None]
    limit = TOL_F32 if io == "f32" else TOL_BF16_OUT
    assert ((whole[pick].double() - exact).abs() / exact.abs().clamp(min=exact.square().mean().sqrt())).max() <= limit
