"""mhcl_post_bwd and mhcl_pre_bwd take one to four waves per token by width, tokens and n: every count
on either side of its lines against the fp64 definition; tolerances as in gpu_harness.py."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for, rel_err, to_np64, TOL_F32, TOL_BF16_OUT

pytestmark = pytest.mark.gpu

# widths of 1, 2, 3 and 4 waves (a row of 16-byte pieces partly filled), tokens around the lines
CASES = [(n, pieces, T, io) for io in ("bf16", "f32") for n, pieces, T in
         ((4, 7, 1024), (4, 7, 1025), (5, 64, 769), (8, 8, 513), (2, 64, 1537), (2, 65, 2000), (2, 128, 16385),
          (3, 128, 16385), (1, 97, 1536), (5, 129, 1100), (6, 192, 1600), (1, 193, 1700), (3, 300, 600))]


@pytest.mark.parametrize("n,pieces,T,io", CASES)
def test_wave_counts_against_fp64(n, pieces, T, io):
    C = (pieces * (8 if io == "bf16" else 4) + 7) // 8 * 8
    wl = si.Workload("waves", n=n, C=C, T=T, io=io, res_mode="subset", n_perm=1)
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=13, device="cuda")
    L = GpuLayer(desc_for(wl, perm=inp["perm"]), inp)
    gen = torch.Generator(device="cuda").manual_seed(1)
    H, Hp, Hq = (torch.rand(t.shape, device="cuda", generator=gen) for t in (L.H_res, L.H_pre, L.H_post))
    mhcl.mhcl_post_bwd(L.d, inp["x"], inp["y"], H, Hq, inp["g_xout"], L.g_x, L.g_y, L.g_H_res, L.g_H_post)
    after_post = L.g_x.clone()
    mhcl.mhcl_pre_bwd(L.d, inp["x"], Hp, inp["g_h"], L.g_x, L.g_H_pre)
    torch.cuda.synchronize()
    x, y, g, gh = (inp[k].double() for k in ("x", "y", "g_xout", "g_h"))
    want = dict(g_y=(Hq.double().unsqueeze(-1) * g).sum(1),
                g_x=after_post.double() + Hp.double().unsqueeze(-1) * gh.unsqueeze(1),
                g_H_post=(g * y.unsqueeze(1)).sum(-1), g_H_pre=(gh.unsqueeze(1) * x).sum(-1),
                g_H_res=torch.stack([(g * x[:, j:j + 1]).sum(-1) for j in range(n)], dim=2))
    after = sum(H.double()[:, i].unsqueeze(-1) * g[:, i:i + 1] for i in range(n))
    out = TOL_F32 if io == "f32" else TOL_BF16_OUT
    assert rel_err(to_np64(after_post), to_np64(after)) <= out
    for k, v in want.items():
        # sums of at most 2400 exact products in fp32, in a tree over lanes: well inside the fp32 bound
        e = rel_err(to_np64(getattr(L, k)), to_np64(v))
        assert e <= (TOL_F32 if k.startswith("g_H") else out), f"{k}: {e:.3e}"
