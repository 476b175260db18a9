"""mhcl_logits with one lane per token (at most 16 logits, many tokens) against the same tokens in batches
that take eight: the same sums in the same order, so the same bits."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import desc_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,mode,K,T", [(1, "lite", 0, 131072), (2, "sk", 0, 131073), (3, "sk", 0, 131327),
                                        (1, "subset", 1, 131100)])
def test_one_lane_per_token_gives_the_same_bits(n, mode, K, T):
    def run(T, inp):
        d = desc_for(si.Workload("logits", n=n, C=64, T=T, res_mode=mode, n_perm=K), perm=inp.get("perm"))
        z, spread = torch.empty(T, d.M, device="cuda"), torch.empty(T, device="cuda")
        mhcl.mhcl_logits(d, inp["x"], inp["W"], inp["b"], inp["alpha"], z, spread,
                         mhcl.binding.new_workspace(d, mhcl.OP_COEFFS))
        return z, spread

    inp = si.make_inputs(si.Workload("logits", n=n, C=64, T=T, res_mode=mode, n_perm=K, backward=False), seed=2,
                         device="cuda")
    z, spread = run(T, inp)
    for t0 in range(0, T, 65536):
        t1 = min(T, t0 + 65536)
        if t1 - t0 < 4096:
            t0 = t1 - 65536     # (few tokens take another projection)
        zb, sb = run(t1 - t0, {**inp, "x": inp["x"][t0:t1].contiguous()})
        assert torch.equal(z[t0:t1], zb) and torch.equal(spread[t0:t1], sb), t0
