"""Pass 1 of the fused backward with the columns split over several blocks per token tile: part counts
that do and do not divide the row, a shorter last part, one step per part, the token counts around
the point where the split ends.  Every token against the oracle; tolerances as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import (GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_BF16_OUT,
                         TOL_BF16_PARAM)

pytestmark = pytest.mark.gpu

# (n, C, T, form): C / 64 column steps, 256 // ceil(T / 64) parts of them (at most 16)
CASES = [(4, 64, 70, "lite"), (4, 320, 64, "lite"), (4, 704, 1000, "lite"), (4, 704, 2049, "sk"),
         (3, 1088, 65, "lite"), (2, 2048, 300, "sk"), (1, 1024, 1, "lite"), (3, 192, 8128, "lite"),
         (3, 192, 8129, "lite"), (4, 128, 16321, "lite")]


@pytest.mark.parametrize("n,C,T,mode", CASES)
def test_column_parts_against_the_oracle(n, C, T, mode):
    wl = si.Workload("parts", n=n, C=C, T=T, res_mode=mode)
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=21, device="cuda")
    ref = oracle_reference(inp, wl)
    L = GpuLayer(desc_for(wl), inp)
    L.backward_fused()
    torch.cuda.synchronize()
    for k, limit in dict(g_x=TOL_BF16_OUT, g_y=TOL_BF16_OUT, g_W=TOL_BF16_PARAM, g_b=TOL_BF16_PARAM,
                         g_alpha=TOL_BF16_PARAM).items():
        e = rel_err(to_np64(getattr(L, k)), ref[k])
        assert e <= limit, f"{k}: {e:.3e} > {limit}"
