"""The bf16 projection where it splits rows into uneven parts (the last one shorter, or with a tail that is no
whole chunk of K steps), against the oracle;
tolerances as in gpu_harness.py."""
import pytest
import torch

import synth_inputs as si
from gpu_harness import GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_BF16_COEF

pytestmark = pytest.mark.gpu


def _wl(n, C, T, mode="lite", K=0):
    return si.Workload(f"n{n}_c{C}_t{T}_{mode}{K}", n=n, C=C, T=T, io="bf16", res_mode=mode, n_perm=K)


CASES = [_wl(4, 1024, 5003),                  # 32 chunks: five parts of six and one of two
         _wl(3, 1472, 2600), _wl(1, 2496, 2501, "sk"),   # 34.5 and 19.5 chunks
         _wl(4, 64, 1300), _wl(2, 64, 2600),  # rows of two and one chunks: one part
         _wl(4, 4160, 1251), _wl(4, 4096, 1409),   # many parts
         _wl(5, 448, 600), _wl(8, 576, 1100, "subset", 40), _wl(6, 704, 1300, "subset", 84)]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_uneven_parts_against_the_oracle(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=23, device="cuda")
    ref = oracle_reference(inp, wl, backward=False)
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    L.forward_separable()
    torch.cuda.synchronize()
    for k in ("H_res", "H_pre", "H_post"):
        e = rel_err(to_np64(getattr(L, k)), ref[k])
        assert e <= TOL_BF16_COEF, f"{k}: {e:.3e}"
