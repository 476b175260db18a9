"""Rows that the full-precision projection splits into parts: the parts' fp64 sums are rounded to fp32 once,
as the sum of a whole row is, so few tokens (up to 16 parts) get the bits they get among 8192 (one
part).  (Orders of fp64 additions differ: a value differs where 2^-53 decides a rounding to 2^-24, 1e-8 of
them.)"""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu
MANY = 8192
PER_TOKEN = ("x", "y", "g_xout", "g_h")


def _wl(n, C, T, io, mode, K):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}{K}", n=n, C=C, T=T, io=io, res_mode=mode, n_perm=K)


def _few(inp, T):
    return {k: (v[:T].contiguous() if k in PER_TOKEN else v) for k, v in inp.items()}


FORMS = [(1, 2048, "f32", "lite", 0), (3, 1920, "f32", "lite", 0), (4, 768, "f32", "lite", 0), (4, 1000, "bf16", "lite", 0),
         (5, 256, "f32", "lite", 0), (2, 1024, "f32", "sk", 0), (5, 264, "f32", "sk", 0), (4, 520, "bf16", "sk", 0),
         (6, 400, "f32", "subset", 60), (8, 264, "bf16", "subset", 128), (8, 128, "f32", "subset", 7)]


@pytest.mark.parametrize("n,C,io,mode,K", FORMS)
def test_split_rows_sum_as_whole_ones(n, C, io, mode, K):
    inp = si.make_inputs(_wl(n, C, MANY, io, mode, K), seed=11, device="cuda")

    def run(T):
        print(f"n={n} C={C} {io} {mode}{K} T={T}", flush=True)
        part = _few(inp, T)
        d = desc_for(_wl(n, C, T, io, mode, K), perm=inp.get("perm"))
        L = GpuLayer(d, part)
        L.forward_fused()
        z, spread = torch.empty(T, d.M, device="cuda"), torch.empty(T, device="cuda")
        mhcl.mhcl_logits(d, part["x"], part["W"], part["b"], part["alpha"], z, spread,
                         mhcl.binding.new_workspace(d, mhcl.OP_COEFFS))
        L.backward_fused()
        torch.cuda.synchronize()
        return dict(H_res=L.H_res, H_pre=L.H_pre, H_post=L.H_post, h=L.h, z=z, spread=spread, g_x=L.g_x, g_y=L.g_y)

    whole = run(MANY)
    for T in (1, 16, 51, 700, 2100):
        for k, v in run(T).items():
            assert torch.equal(v, whole[k][:T]), (T, k, int((v != whole[k][:T]).sum()))


@pytest.mark.parametrize("n,C,mode,K", [(4, 1024, "lite", 0), (2, 4096, "sk", 0), (5, 256, "lite", 0), (6, 320, "subset", 30)])
def test_split_bf16_rows_sum_as_whole_f32_ones(n, C, mode, K):
    """Few bf16 tokens at C a multiple of 64, whose larger batches take another projection."""
    inp = si.make_inputs(_wl(n, C, 16, "bf16", mode, K), seed=12, device="cuda")
    out = []
    for io, copies in (("bf16", 1), ("f32", MANY // 16)):
        x = inp["x"].to(torch.float32 if io == "f32" else torch.bfloat16).repeat(copies, *[1] * (inp["x"].dim() - 1))
        d = desc_for(_wl(n, C, 16 * copies, io, mode, K), perm=inp.get("perm"))
        z, spread = torch.empty(16 * copies, d.M, device="cuda"), torch.empty(16 * copies, device="cuda")
        mhcl.mhcl_logits(d, x, inp["W"], inp["b"], inp["alpha"], z, spread,
                         mhcl.binding.new_workspace(d, mhcl.OP_COEFFS))
        out.append((z[:16], spread[:16]))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
