"""Rows that the full-precision projection splits into 32 parts (a block or two of tokens), and the last token count that
does, against the oracle, behind each stage that adds the slices; tolerances as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import (GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_BF16_COEF, TOL_BF16_OUT,
                         TOL_BF16_PARAM, TOL_F32)

pytestmark = pytest.mark.gpu


def _wl(n, C, T, io="bf16", mode="lite", K=0):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}{K}", n=n, C=C, T=T, io=io, res_mode=mode, n_perm=K)


CASES = [_wl(4, 4096, 1), _wl(4, 4096, 32), _wl(4, 4096, 33), _wl(4, 4096, 17, mode="sk"), _wl(5, 2048, 16),
         _wl(5, 2048, 31, mode="sk"), _wl(8, 2048, 30, "bf16", "subset", 64), _wl(5, 2048, 18, "f32"), _wl(4, 4104, 5, "f32")]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_rows_in_many_parts(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=43, device="cuda")
    ref = oracle_reference(inp, wl)
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    out, coef, par = ((TOL_F32,) * 3 if wl.io == "f32" else (TOL_BF16_OUT, TOL_BF16_COEF, TOL_BF16_PARAM))
    tol = dict(H_res=coef, H_pre=coef, H_post=coef, h=out, x_out=out, g_x=out, g_y=out, g_W=par, g_b=par, g_alpha=par)
    both = [(L.forward_separable, L.backward_separable)]
    if wl.io == "f32" or wl.n > 4:   # (the fused backward of narrow bf16 rows has no part in this: another projection)
        both.append((L.forward_fused, L.backward_fused))
    for calls in both:
        for call in calls:
            call()
        torch.cuda.synchronize()
        for k, limit in tol.items():
            e = rel_err(to_np64(getattr(L, k)), ref[k])
            assert e <= limit, f"{calls[1].__name__} {k}: {e:.3e} > {limit}"
