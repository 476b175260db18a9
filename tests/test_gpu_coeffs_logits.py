"""mhcl_coeffs_logits against the oracle where the per-token stage writes the logits itself (each lane count, edges of
its blocks), where a launch of its own does, and behind each kind of slices; tolerances as in gpu_harness.py and
test_gpu_diag.py."""
import pytest
import torch

import oracle
import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import desc_for, rel_err, to_np64, TOL_BF16_COEF, TOL_F32

pytestmark = pytest.mark.gpu


def _wl(n, C, T, io="bf16", mode="lite", K=0):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}{K}", n=n, C=C, T=T, io=io, res_mode=mode, n_perm=K, backward=False)


CASES = [_wl(4, 64, 1), _wl(4, 128, 1251, mode="sk"), _wl(3, 64, 2533), _wl(2, 64, 33, "f32", "sk"), _wl(1, 64, 31, "f32"),
         _wl(4, 64, 16385, mode="sk"), _wl(5, 64, 601, mode="sk"), _wl(4, 1024, 40, "f32"),   # lanes; fp64 slices
         _wl(1, 64, 200001), _wl(5, 128, 600), _wl(5, 1024, 40, "f32"), _wl(7, 64, 70, "bf16", "subset", 20)]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_coefficients_and_logits_in_one_call(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=29, device="cuda")
    d = desc_for(wl, perm=inp.get("perm"))
    e = lambda *s: torch.full(s, float("nan"), device="cuda")  # noqa: E731
    H, Hp, Hq, z, spread = e(wl.T, wl.n, wl.n), e(wl.T, wl.n), e(wl.T, wl.n), e(wl.T, d.M), e(wl.T)
    mhcl.mhcl_coeffs_logits(d, inp["x"], inp["W"], inp["b"], inp["alpha"], H, Hp, Hq, z, spread,
                            mhcl.binding.new_workspace(d, mhcl.OP_COEFFS))
    torch.cuda.synchronize()
    x, y = inp["x"], inp.get("y", inp["x"][:, 0])
    f = {k: to_np64(inp[k]) for k in ("W", "b", "alpha")}
    sigma = inp["perm"].cpu().numpy().astype("int32") if wl.res_mode == "subset" else None
    ref = oracle.forward(to_np64(x), f["W"], f["b"], f["alpha"], to_np64(y), eps=wl.eps, res_mode=wl.res_mode,
                         iters=wl.sk_iters, sigma=sigma)
    coef, logit = (TOL_F32, 1e-5) if wl.io == "f32" else (TOL_BF16_COEF, 3e-5)
    for k, got in dict(H_res=H, H_pre=Hp, H_post=Hq).items():
        assert rel_err(to_np64(got), ref[k]) <= coef, k
    # the same logits as the call that writes only them, which test_gpu_diag.py holds against the oracle
    z2, spread2 = torch.empty_like(z), torch.empty_like(spread)
    mhcl.mhcl_logits(d, inp["x"], inp["W"], inp["b"], inp["alpha"], z2, spread2,
                     mhcl.binding.new_workspace(d, mhcl.OP_COEFFS))
    torch.cuda.synchronize()
    assert rel_err(to_np64(z), to_np64(z2)) <= logit and rel_err(to_np64(spread), to_np64(spread2)) <= logit
