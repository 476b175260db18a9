"""Infinities and NaN reach what depends on them and nothing else: not through the lanes of a token's group
that own no logit, nor through the padding tokens of a block."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu

CASES = [(4, "lite", 0, 70), (2, "lite", 0, 1), (3, "sk", 0, 33), (1, "sk", 0, 5), (5, "sk", 0, 31),
         (5, "lite", 0, 70), (6, "subset", 20, 33), (4, "lite", 0, 16385)]


def _grads(wl, inp):
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    out = {}
    for calls in ((L.backward_fused,), (L.forward_separable, L.backward_separable)):
        for call in calls:
            call()
        torch.cuda.synchronize()
        out[calls[-1].__name__] = (L.g_b.clone(), L.g_alpha.clone())
    return out


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("n,mode,K,T", CASES)
def test_a_gate_that_is_not_finite_leaves_the_other_sums_alone(n, mode, K, T, io):
    wl = si.Workload("nonfinite", n=n, C=64, T=T, io=io, res_mode=mode, n_perm=K)
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=9, device="cuda")
    R = wl.M - 2 * n
    # the first pre gate and the last post gate: logit and alpha it belongs to
    for col, group in ((R, 1), (wl.M - 1, 2)):
        W, want = inp["W"], None
        for value in (1e30, float("inf"), float("nan")):     # 1e30: the gate at its limit, all sums finite
            inp["W"] = W.clone()
            inp["W"][7, col] = value
            got = _grads(wl, inp)
            want = want or got
            for call in got:
                (b0, a0), (b1, a1) = want[call], got[call]
                others = torch.arange(wl.M, device="cuda") != col
                if call == "backward_fused":     # (the separable calls' x_out and g_H depend on every gate)
                    assert torch.equal(b0[others], b1[others]), (call, col, value)
                for g in range(3):
                    if g != group:
                        assert torch.isfinite(a1[g]) and torch.equal(a0[g], a1[g]), (call, col, value, g)
        inp["W"] = W


@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_an_infinite_gradient_on_one_permutation(io):
    """n = 2: g_a = (inf, finite), <a, g_a> = inf, so g_z = a (g_a - <a, g_a>) = (NaN, -inf)."""
    wl = si.Workload("inf", n=2, C=64, T=1, io=io)
    inp = si.make_inputs(wl, seed=9, device="cuda")
    L = GpuLayer(desc_for(wl), inp)
    for t in (L.g_H_res, L.g_H_pre, L.g_H_post, L.g_x):
        t.fill_(0.5)
    L.g_H_res[0, 0, 0] = float("inf")
    mhcl.mhcl_coeffs_bwd(L.d, inp["x"], inp["W"], inp["b"], inp["alpha"], L.g_H_res, L.g_H_pre, L.g_H_post,
                         L.g_x, L.g_W, L.g_b, L.g_alpha, L.ws)
    torch.cuda.synchronize()
    assert torch.isnan(L.g_b[0]) and L.g_b[1] == -float("inf") and torch.isfinite(L.g_b[2:]).all()
