"""The full-precision projection at rows of one to three steps (one wave per 16 tokens up to two of them)
with four to nine logit tiles, a row without steps for its last part, against the oracle; tolerances
as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_F32, TOL_BF16_OUT, TOL_BF16_COEF

pytestmark = pytest.mark.gpu


def _wl(n, C, T, io, mode="lite", K=0):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}{K}", n=n, C=C, T=T, io=io, res_mode=mode, n_perm=K)


CASES = [_wl(5, 8, 17, "bf16"), _wl(5, 8, 131, "f32"), _wl(4, 8, 33, "f32", "subset", 24), _wl(4, 16, 15, "bf16", "subset", 24),
         _wl(6, 8, 50, "bf16", "subset", 60), _wl(8, 8, 100, "bf16", "subset", 100), _wl(8, 8, 64, "f32", "subset", 70),
         _wl(8, 16, 16, "bf16", "subset", 64), _wl(7, 8, 1, "bf16", "subset", 128),
         _wl(2, 2064, 33, "bf16")]   # 129 steps in 16 parts of nine: the last part has none


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_short_rows_against_the_oracle(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=17, device="cuda")
    ref = oracle_reference(inp, wl, backward=False)
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    L.forward_fused()
    torch.cuda.synchronize()
    out, coef = (TOL_F32, TOL_F32) if wl.io == "f32" else (TOL_BF16_OUT, TOL_BF16_COEF)
    for k, limit in dict(H_res=coef, H_pre=coef, H_post=coef, h=out).items():
        e = rel_err(to_np64(getattr(L, k)), ref[k])
        assert e <= limit, f"{k}: {e:.3e} > {limit}"
