"""The two passes of the bf16 backward for n <= 4 with W as it is (up to 4096 tokens; the permutation form at n = 3
up to 2^20 tokens times columns) and packed, and the sums behind g_b and
g_alpha in pass 2's launch (one chunk of tokens) or after it, against the oracle: logits that fill their tiles, end
inside a group of eight, or need scalar loads; tolerances as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_BF16_OUT, TOL_BF16_PARAM

pytestmark = pytest.mark.gpu


def _wl(n, C, T, mode="lite"):
    return si.Workload(f"n{n}_c{C}_t{T}_{mode}", n=n, C=C, T=T, io="bf16", res_mode=mode)


CASES = [_wl(1, 64, 1), _wl(1, 192, 65, "sk"), _wl(2, 64, 64), _wl(2, 128, 63, "sk"), _wl(3, 64, 66), _wl(3, 320, 129, "sk"),
         _wl(4, 64, 64), _wl(4, 128, 65), _wl(4, 64, 200, "sk"), _wl(4, 1024, 40), _wl(4, 64, 4096), _wl(4, 64, 4097),
         _wl(2, 64, 4096), _wl(3, 128, 1024), _wl(3, 128, 1025, "sk"), _wl(3, 1024, 1024), _wl(3, 1024, 1025), _wl(3, 64, 4096),
         _wl(3, 64, 4097), _wl(3, 192, 4096, "sk"), _wl(3, 192, 4097, "sk"), _wl(1, 2048, 300), _wl(3, 1024, 1)]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_fused_backward_against_the_oracle(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=41, device="cuda")
    ref = oracle_reference(inp, wl)
    L = GpuLayer(desc_for(wl), inp)
    names = dict(g_x=TOL_BF16_OUT, g_y=TOL_BF16_OUT, g_W=TOL_BF16_PARAM, g_b=TOL_BF16_PARAM, g_alpha=TOL_BF16_PARAM)
    for k in names:
        getattr(L, k).fill_(float("nan"))
    L.backward_fused()
    torch.cuda.synchronize()
    for k, limit in names.items():
        e = rel_err(to_np64(getattr(L, k)), ref[k])
        assert e <= limit, f"{k}: {e:.3e} > {limit}"
