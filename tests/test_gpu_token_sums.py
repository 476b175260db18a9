"""Sums over tokens (g_b, g_alpha) are pairwise inside a block of tokens.  With identical tokens every
partial sum of 2^k of them is exact in a pairwise order, so g_b and g_alpha of T tokens must be T times
those of the first token alone (the others with zero gradients), rounded once: no tolerance.  (One
after the other, 3 v, 5 v, 7 v ... round.)"""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu

CASES = [(4, "lite", 0), (3, "sk", 0), (1, "lite", 0), (5, "sk", 0), (5, "lite", 0), (6, "subset", 20)]


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("T", [32, 48, 64, 16384])
@pytest.mark.parametrize("n,mode,K", CASES)
def test_sums_of_identical_tokens_are_exact(n, mode, K, T, io):
    wl = si.Workload("sums", n=n, C=64, T=T, io=io, res_mode=mode, n_perm=K)
    print(f"case {wl}", flush=True)
    one = si.make_inputs(si.Workload("one", n=n, C=64, T=1, io=io, res_mode=mode, n_perm=K), seed=3, device="cuda")
    inp = {k: (v.expand(T, *v.shape[1:]).contiguous() if k in ("x", "y", "g_xout", "g_h") else v)
           for k, v in one.items()}
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    g_H = [torch.linspace(-1, 1, t[0].numel(), device="cuda").view(t[0].shape).expand_as(t).contiguous()
           for t in (L.g_H_res, L.g_H_pre, L.g_H_post)]

    def sums():
        L.backward_fused()
        fused = L.g_b.clone(), L.g_alpha.clone()
        L.g_x.zero_()
        mhcl.mhcl_coeffs_bwd(L.d, inp["x"], inp["W"], inp["b"], inp["alpha"], *g_H, L.g_x, L.g_W, L.g_b,
                             L.g_alpha, L.ws)
        return fused + (L.g_b.clone(), L.g_alpha.clone())

    every = sums()
    for t in [inp["g_xout"], inp["g_h"]] + g_H:
        t[1:].zero_()
    first = sums()
    for name, a, v in zip(("fused g_b", "fused g_alpha", "coeffs g_b", "coeffs g_alpha"), every, first):
        assert torch.equal(a, (v.double() * T).float()), name
