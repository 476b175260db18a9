"""The per-token stage against the oracle at the edges of its blocks (32 or 64 tokens, four, eight
or sixteen lanes per token): every n and form, Sinkhorn-Knopp iteration counts from one to the
largest (whose divisors take the most LDS), and the token count at which the lanes per token
change.  C = 64 keeps the rest small.  Tolerances as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import (GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_F32, TOL_BF16_OUT,
                         TOL_BF16_COEF, TOL_BF16_PARAM)

pytestmark = pytest.mark.gpu

CASES = [(n, T, mode, 20, io) for n in (1, 2, 3, 4) for mode in ("lite", "sk")
         for T, io in ((1, "bf16"), (33, "f32"), (65, "bf16"))]
CASES += [(5, 31, "sk", 32, "bf16"), (5, 65, "sk", 20, "f32"), (4, 95, "sk", 32, "bf16"), (4, 32, "sk", 1, "f32"),
          (3, 64, "sk", 32, "f32"),
          (4, 16383, "lite", 0, "bf16"), (4, 16384, "lite", 0, "bf16"), (3, 16385, "lite", 0, "bf16"),
          (2, 16447, "sk", 20, "bf16"), (4, 16384, "sk", 20, "bf16"), (1, 16449, "lite", 0, "f32")]


@pytest.mark.parametrize("n,T,mode,iters,io", CASES)
def test_token_stage_against_the_oracle(n, T, mode, iters, io):
    wl = si.Workload("stage", n=n, C=64, T=T, io=io, res_mode=mode, sk_iters=iters or 20, alpha=(1.5, 0.7, 1.2))
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=5, device="cuda")
    ref = oracle_reference(inp, wl)
    L = GpuLayer(desc_for(wl), inp)
    out, coef, par = ((TOL_F32,) * 3 if io == "f32" else (TOL_BF16_OUT, TOL_BF16_COEF, TOL_BF16_PARAM))
    tol = dict(H_res=coef, H_pre=coef, H_post=coef, h=out, x_out=out, g_x=out, g_y=out, g_W=par, g_b=par,
               g_alpha=par)
    for calls in ((L.forward_fused, L.backward_fused), (L.forward_separable, L.backward_separable)):
        for call in calls:
            call()
        torch.cuda.synchronize()
        for k, limit in tol.items():
            e = rel_err(to_np64(getattr(L, k)), ref[k])
            assert e <= limit, f"{calls[1].__name__} {k}: {e:.3e} > {limit}"
