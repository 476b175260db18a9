"""A workspace made for a larger batch serves a smaller one, with the results of one made for it."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu

# (n, C, io, form, K, large T, small T): the small batch splits its rows or columns more often
CASES = [(4, 768, "f32", "lite", 0, 8192, 8176), (4, 4096, "f32", "lite", 0, 1024, 1008), (4, 64, "bf16", "lite", 0, 32784, 32768),
         (3, 1024, "bf16", "sk", 0, 16400, 300), (5, 320, "bf16", "lite", 0, 560, 500), (8, 128, "bf16", "subset", 64, 1100, 900),
         (4, 1000, "bf16", "lite", 0, 9000, 100)]


@pytest.mark.parametrize("n,C,io,mode,K,large,small", CASES)
def test_a_larger_batch_s_workspace(n, C, io, mode, K, large, small):
    form = dict(n=n, C=C, io=io, res_mode=mode, n_perm=K)
    wl = si.Workload("small", T=small, **form)
    print(f"case {wl} in the workspace of {large} tokens", flush=True)
    inp = si.make_inputs(wl, seed=23, device="cuda")
    names = ("H_res", "H_pre", "H_post", "h", "x_out", "g_x", "g_y", "g_W", "g_b", "g_alpha")
    d = desc_for(wl, perm=inp.get("perm"))
    big = desc_for(si.Workload("large", T=large, **form), perm=inp.get("perm"))

    def outputs(ws_of):
        L = GpuLayer(d, inp)
        out = []
        for calls, ops in (((L.forward_fused, L.backward_fused), (mhcl.OP_FWD_COEFFS_PRE, mhcl.OP_BWD_FUSED)),
                           ((L.forward_separable, L.backward_separable), (mhcl.OP_COEFFS, mhcl.OP_COEFFS_BWD))):
            for call, op in zip(calls, ops):
                L.ws = ws_of(op)
                call()
            out += [getattr(L, k).clone() for k in names]
        torch.cuda.synchronize()
        return out

    own = outputs(lambda op: torch.full((mhcl.workspace_bytes(d, op),), 255, dtype=torch.uint8, device="cuda"))
    # (bytes past the large size stay as they are)
    kept = []

    def shared(op):
        nb = mhcl.workspace_bytes(big, op)
        kept.append((nb, torch.full((nb + 4096,), 255, dtype=torch.uint8, device="cuda")))
        return kept[-1][1][:nb]

    for a, b in zip(own, outputs(shared)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert all((t[nb:] == 255).all() for nb, t in kept)
