"""The fused backward (bf16) where pass 1 holds two tiles per wave and where pass 2 gives a compute unit one 64-column
step: one iteration or three of them, odd and even numbers of steps, the last block short, against the oracle;
tolerances as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_BF16_OUT, TOL_BF16_PARAM

pytestmark = pytest.mark.gpu


def _wl(n, C, T, mode="lite"):
    return si.Workload(f"n{n}_c{C}_t{T}_{mode}", n=n, C=C, T=T, io="bf16", res_mode=mode)


CASES = [_wl(4, 768, 1344), _wl(4, 768, 1345), _wl(4, 768, 2689, "sk"), _wl(4, 768, 4033),   # 1, 1 x 2, 3, 2 x 2 iterations
         _wl(3, 192, 131), _wl(2, 1088, 1000, "sk"), _wl(1, 64, 1), _wl(4, 128, 64), _wl(3, 1024, 1025)]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_few_tokens_against_the_oracle(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=31, device="cuda")
    ref = oracle_reference(inp, wl)
    L = GpuLayer(desc_for(wl), inp)
    L.backward_fused()
    torch.cuda.synchronize()
    for k, limit in dict(g_x=TOL_BF16_OUT, g_y=TOL_BF16_OUT, g_W=TOL_BF16_PARAM, g_b=TOL_BF16_PARAM,
                         g_alpha=TOL_BF16_PARAM).items():
        e = rel_err(to_np64(getattr(L, k)), ref[k])
        assert e <= limit, f"{k}: {e:.3e} > {limit}"
