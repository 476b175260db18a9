"""Equal tokens of one call get equal coefficients, logits and h wherever they stand in the batch, in every bit: a token's
sums are added in an order that does not depend on its place.  Rows long enough to be walked in many chunks and in
one or more parts, whole and ragged, batches of several blocks of either projection."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu


def _wl(n, C, T, mode="lite", K=0, io="bf16"):
    return si.Workload(f"n{n}_c{C}_t{T}_{mode}{K}" + ("_f32" if io == "f32" else ""), n=n, C=C, T=T, io=io, res_mode=mode,
                       n_perm=K, backward=False)


CASES = [_wl(4, 64, 3000), _wl(4, 256, 5000), _wl(4, 1024, 2048), _wl(4, 1024, 40000), _wl(3, 1472, 2600), _wl(1, 2496, 2700, "sk"),
         _wl(4, 4096, 1409), _wl(4, 768, 3001, "sk"), _wl(5, 448, 1000), _wl(8, 1024, 5000, "subset", 64),
         # the fp64 projection in parts and whole, one token per lane
         _wl(4, 4096, 100), _wl(6, 512, 300, "subset", 100), _wl(4, 768, 3000, io="f32"), _wl(3, 200, 20000, "sk", io="f32"),
         _wl(2, 64, 70000, "sk")]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_equal_tokens(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=37, device="cuda")
    distinct = 7   # (no divisor of a block: every token stands at every place of one)
    inp["x"] = inp["x"][:distinct].repeat(-(-wl.T // distinct), 1, 1)[:wl.T].contiguous()
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    z = torch.empty(wl.T, wl.M, device="cuda")
    spread = torch.empty(wl.T, device="cuda")
    L.forward_fused()
    got = {f"fused {k}": getattr(L, k).clone() for k in ("H_res", "H_pre", "H_post", "h")}
    mhcl.mhcl_coeffs_logits(L.d, inp["x"], inp["W"], inp["b"], inp["alpha"], L.H_res, L.H_pre, L.H_post, z, spread,
                            mhcl.binding.new_workspace(L.d, mhcl.OP_COEFFS))
    got.update({"H_res": L.H_res, "H_pre": L.H_pre, "H_post": L.H_post, "z": z, "spread": spread})
    torch.cuda.synchronize()
    for k, v in got.items():
        first = v[:distinct].repeat(-(-wl.T // distinct), *([1] * (v.dim() - 1)))[:wl.T]
        moved = int((v != first).sum())
        assert moved == 0, f"{k}: {moved} values depend on the token's place"
