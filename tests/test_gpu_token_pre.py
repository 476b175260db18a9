"""mhcl_fwd_coeffs_pre where one launch takes the coefficients and h, against the separate calls, which test_gpu_parity.py
holds against the oracle: each lane count, blocks whose chunks of h start and end inside rows, rows of one chunk,
gates that one thread adds (many tokens a block) and ones that many stage, both sides of the rule's lines.
Either computes the same sums in the same order and the same products fused, so the results are the same in every bit."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu


def _wl(n, C, T, io="bf16", mode="lite", K=0):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}{K}", n=n, C=C, T=T, io=io, res_mode=mode, n_perm=K, backward=False)


CASES = [_wl(4, 4096, 1), _wl(4, 4096, 17), _wl(3, 200, 7), _wl(4, 768, 683), _wl(2, 8, 1030), _wl(1, 8, 511, "f32"),
         _wl(4, 72, 2049, "f32"), _wl(4, 1024, 5120), _wl(4, 1024, 5121), _wl(4, 64, 16384), _wl(2, 128, 20011),
         _wl(4, 768, 3001, mode="sk"), _wl(5, 136, 333, mode="sk"), _wl(1, 64, 70000, mode="sk"),
         _wl(5, 1024, 16), _wl(5, 64, 65, "f32"), _wl(8, 512, 33, "bf16", "subset", 30), _wl(8, 8, 700, "bf16", "subset", 100),
         _wl(6, 256, 2000, "f32", "subset", 20), _wl(7, 64, 3000, "bf16", "subset", 128),
         # fp64 slices: both sides of the line, bf16 and f32
         _wl(4, 1288, 4070), _wl(4, 1288, 4071), _wl(3, 1288, 2035, "f32"), _wl(3, 1288, 2036, "f32"), _wl(4, 3072, 4096, "f32"),
         _wl(4, 3072, 4097, "f32"),
         # more than 64 permutations: one launch for few tokens only
         _wl(8, 64, 8192, "bf16", "subset", 65), _wl(8, 64, 8193, "bf16", "subset", 65), _wl(6, 512, 8192, "bf16", "subset", 80),
         _wl(6, 520, 8192, "bf16", "subset", 80), _wl(6, 512, 20000, "bf16", "subset", 64)]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_h_of_the_fused_call(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=31, device="cuda")
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    for k in ("H_res", "H_pre", "H_post", "h"):
        getattr(L, k).fill_(float("nan"))
    mhcl.mhcl_fwd_coeffs_pre(L.d, inp["x"], inp["W"], inp["b"], inp["alpha"], L.H_res, L.H_pre, L.H_post, L.h,
                             mhcl.binding.new_workspace(L.d, mhcl.OP_FWD_COEFFS_PRE))
    got = {k: getattr(L, k).clone() for k in ("H_res", "H_pre", "H_post", "h")}
    mhcl.mhcl_coeffs(L.d, inp["x"], inp["W"], inp["b"], inp["alpha"], L.H_res, L.H_pre, L.H_post,
                     mhcl.binding.new_workspace(L.d, mhcl.OP_COEFFS))
    mhcl.mhcl_pre(L.d, inp["x"], L.H_pre, L.h)
    torch.cuda.synchronize()
    for k in got:
        other = int((got[k] != getattr(L, k)).sum())
        assert other == 0, f"{k}: {other} values differ"
