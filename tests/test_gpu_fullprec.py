"""The full-precision matrix-core kernels (f32 streams, widths that are no multiple of 64, the
separable backward) against the oracle at the edges of their tiles: column counts around the 64 and
128 columns of a wave, token counts around the 4-token groups, the 64- and 128-token steps and the
token chunks, one to nine logit tiles.  Tolerances as in gpu_harness.py (f32 streams 1e-5)."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import (GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_F32, TOL_BF16_OUT,
                         TOL_BF16_COEF, TOL_BF16_PARAM)

pytestmark = pytest.mark.gpu


def _wl(n, C, T, io, mode="lite", K=0):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}{K}", n=n, C=C, T=T, io=io, res_mode=mode, n_perm=K)


CASES = [
    _wl(1, 8, 1, "f32"), _wl(1, 8, 5, "bf16"),                 # one partial column tile, one partial token group
    _wl(2, 24, 127, "f32"), _wl(4, 16, 129, "f32"),            # one column block exactly full, a step plus one token
    _wl(4, 72, 511, "bf16"), _wl(3, 40, 513, "f32"),           # ragged last column block, two token chunks
    _wl(4, 64, 257, "bf16"), _wl(4, 1000, 300, "bf16"),
    _wl(4, 136, 2049, "f32"), _wl(5, 104, 260, "f32"),         # nine token chunks; nine logit tiles
    _wl(5, 64, 70, "bf16", "sk"), _wl(8, 40, 33, "f32", "subset", 20),
    # widths that are multiples of 64: the last token count of the fp64 projection, the first of the
    # bf16 one with its row split four ways
    _wl(4, 1024, 1250, "bf16"), _wl(4, 1024, 1251, "bf16"), _wl(5, 320, 555, "bf16"), _wl(5, 320, 556, "bf16"),
    _wl(8, 128, 1001, "bf16", "subset", 64), _wl(4, 4096, 1300, "bf16"), _wl(7, 64, 700, "bf16", "subset", 50),
    _wl(5, 64, 900, "bf16", "sk"), _wl(2, 64, 2501, "bf16"), _wl(3, 64, 16, "bf16", "sk"), _wl(2, 4096, 3, "bf16"),
    _wl(7, 56, 131, "bf16", "subset", 50), _wl(8, 24, 64, "f32", "subset", 111),
]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_edges_against_the_oracle(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=11, device="cuda")
    ref = oracle_reference(inp, wl)
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    out, coef, par = ((TOL_F32,) * 3 if wl.io == "f32" else (TOL_BF16_OUT, TOL_BF16_COEF, TOL_BF16_PARAM))
    tol = dict(H_res=coef, H_pre=coef, H_post=coef, h=out, x_out=out, g_x=out, g_y=out, g_W=par, g_b=par,
               g_alpha=par)
    for calls in ((L.forward_fused, L.backward_fused), (L.forward_separable, L.backward_separable)):
        for call in calls:
            call()
        torch.cuda.synchronize()
        for k, limit in tol.items():
            e = rel_err(to_np64(getattr(L, k)), ref[k])
            assert e <= limit, f"{calls[1].__name__} {k}: {e:.3e} > {limit}"
