"""mhcl_fwd_coeffs_pre and its static variant against mhcl_coeffs followed by mhcl_pre, bit for bit, wherever they take the same
projection: one launch for the coefficients and h must give what the two give, in every lane count, form and
stream type, with one part of a row or several, and h is H_pre x of the H_pre returned."""
import random

import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu


def _wl(n, C, T, io="bf16", mode="lite", K=0):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}{K}", n=n, C=C, T=T, io=io, res_mode=mode, n_perm=K, backward=False)


def _drawn(seed, count):
    rng, out = random.Random(seed), []
    while len(out) < count:
        mode = rng.choice(["lite", "lite", "sk", "sk", "subset"])
        n = rng.randint(1, 8 if mode == "subset" else 5)
        K = rng.randint(1, min(128, [1, 2, 6, 24, 120][n - 1] if n <= 5 else 128)) if mode == "subset" else 0
        io = rng.choice(["bf16", "bf16", "f32"])
        C = rng.choice([8 * rng.randint(1, 64), 64 * rng.randint(1, 32)])
        T = int(2 ** rng.uniform(0, 13.5))
        if n * C * T <= 2 ** 25:
            out.append(_wl(n, C, T, io, mode, K))
    return out


CASES = [_wl(4, 4096, 1), _wl(4, 4096, 17), _wl(4, 4096, 1409), _wl(4, 1024, 5003), _wl(4, 64, 16384), _wl(4, 64, 30000, mode="sk"),
         _wl(4, 768, 3001, mode="sk"), _wl(5, 136, 333, mode="sk"), _wl(5, 1024, 16), _wl(5, 320, 3000), _wl(2, 8, 1030),
         _wl(8, 512, 33, "bf16", "subset", 30), _wl(7, 64, 3000, "bf16", "subset", 128), _wl(3, 200, 777, "f32")]


@pytest.mark.parametrize("wl", CASES + _drawn(7, 40), ids=lambda w: w.name)
def test_same_bits(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=41, device="cuda")
    L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
    args = (L.d, inp["x"], inp["W"], inp["b"], inp["alpha"], L.H_res, L.H_pre, L.H_post)
    names = ("H_res", "H_pre", "H_post", "h")

    def of(call):
        for k in names:
            getattr(L, k).fill_(float("nan"))
        call()
        return {k: getattr(L, k).clone() for k in names}

    def separate():
        mhcl.mhcl_coeffs(*args, L.ws)
        mhcl.mhcl_pre(L.d, inp["x"], L.H_pre, L.h)

    want = of(separate)
    assert all(bool(torch.isfinite(v.float()).all()) for v in want.values())
    for name, call in (("fused", lambda: mhcl.mhcl_fwd_coeffs_pre(*args, L.h, L.ws)),
                       ("static", lambda: mhcl.mhcl_fwd_coeffs_pre_static(*args, L.h))):
        got = of(call)
        for k in names:
            other = int((got[k] != want[k]).sum())
            assert other == 0, f"{name} {k}: {other} values differ"
