"""The per-token stage with one token per lane (many tokens; Sinkhorn-Knopp, and the forward of the
permutation form) against the same tokens in batches of a few
thousand, which take the lane groups that test_gpu_token_stage.py checks against the oracle: per-token
outputs batch by batch, sums over tokens added in fp64.  Both sides round alike up to the order of
fp32 sums and, in bf16 streams, single bf16 steps; tolerances as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import (GpuLayer, desc_for, rel_err, to_np64, TOL_F32, TOL_BF16_OUT, TOL_BF16_COEF,
                         TOL_BF16_PARAM)

pytestmark = pytest.mark.gpu

# (n, T, iterations (0: permutation form), io): from the first count at which both directions take one token per lane; partly filled blocks
CASES = [(1, 45000, 32, "bf16"), (2, 43751, 32, "bf16"), (3, 47563, 32, "bf16"), (4, 137501, 32, "bf16"),
         (5, 23750, 32, "bf16"), (5, 33999, 20, "bf16"), (1, 200001, 1, "bf16"), (3, 47501, 32, "f32"), (1, 200000, 0, "bf16"), (2, 200193, 0, "f32"),
         (3, 200063, 0, "bf16"), (4, 200001, 0, "bf16")]
BATCH = 5120


@pytest.mark.parametrize("n,T,iters,io", CASES)
def test_one_token_per_lane_against_smaller_batches(n, T, iters, io):
    form = dict(n=n, C=64, io=io, res_mode="sk" if iters else "lite", sk_iters=iters or 20)
    wl = si.Workload("many", T=T, alpha=(1.5, 0.7, 1.2), **form)
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=5, device="cuda")
    out, coef, par = ((TOL_F32,) * 3 if io == "f32" else (TOL_BF16_OUT, TOL_BF16_COEF, TOL_BF16_PARAM))
    per_token = dict(H_res=coef, H_pre=coef, H_post=coef, h=out, x_out=out, g_x=out, g_y=out)
    L = GpuLayer(desc_for(wl), inp)
    L.step()
    sums = {k: 0.0 for k in ("g_W", "g_b", "g_alpha")}
    for t0 in range(0, T, BATCH):
        part = {k: (v[t0:t0 + BATCH].contiguous() if k in ("x", "y", "g_xout", "g_h") else v) for k, v in inp.items()}
        t1 = min(T, t0 + BATCH)
        B = GpuLayer(desc_for(si.Workload("batch", T=t1 - t0, **form)), part)
        B.step()
        for k, limit in per_token.items():
            e = rel_err(to_np64(getattr(L, k)[t0:t1]), to_np64(getattr(B, k)))
            assert e <= limit, f"{k} from token {t0}: {e:.3e} > {limit}"
        for k in sums:
            sums[k] = sums[k] + getattr(B, k).double()
    for k, want in sums.items():
        e = rel_err(to_np64(getattr(L, k)), to_np64(want))
        assert e <= par, f"{k}: {e:.3e} > {par}"
