"""The backward's launches with blocks of two or three roles, against the oracle: one to four waves per token in the dot
products' role (three leave two of a block's waves idle), tokens that fill its last block or not, one token chunk of
g_W and several, each n and number of logit tiles, both stream types; tolerances as in gpu_harness.py."""
import ctypes

import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from bench import HipEvents
from gpu_harness import (GpuLayer, desc_for, oracle_reference, rel_err, to_np64, TOL_BF16_OUT,
                         TOL_BF16_PARAM, TOL_F32)

pytestmark = pytest.mark.gpu


def _wl(n, C, T, io="f32", mode="lite"):
    return si.Workload(f"n{n}_c{C}_t{T}_{io}_{mode}", n=n, C=C, T=T, io=io, res_mode=mode)


CASES = [_wl(1, 8, 9), _wl(2, 264, 35), _wl(3, 520, 7), _wl(4, 776, 17), _wl(4, 768, 300), _wl(4, 64, 257),
         _wl(5, 520, 3, mode="sk"), _wl(5, 1032, 33, mode="sk"), _wl(1, 520, 513, mode="sk"),
         _wl(4, 1032, 5, "bf16"), _wl(4, 1544, 301, "bf16"), _wl(3, 2056, 65, "bf16", "sk"), _wl(5, 72, 530, "bf16", "sk"),
         _wl(2, 1032, 1, "bf16"),
         # both sides of the line up to which the projection and the dot products share a launch
         _wl(5, 40, 800, "bf16", "sk"), _wl(5, 40, 801, "bf16", "sk"), _wl(5, 8, 16384, mode="sk"), _wl(5, 8, 16385, mode="sk"),
         _wl(4, 8, 10240), _wl(4, 8, 10241, "bf16"), _wl(3, 8, 10240, "bf16"), _wl(3, 8, 10241), _wl(2, 8, 131073), _wl(1, 8, 131073, mode="sk")]


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_joint_launches_against_the_oracle(wl):
    print(f"case {wl}", flush=True)
    inp = si.make_inputs(wl, seed=37, device="cuda")
    ref = oracle_reference(inp, wl)
    L = GpuLayer(desc_for(wl), inp)
    out, par = (TOL_F32, TOL_F32) if wl.io == "f32" else (TOL_BF16_OUT, TOL_BF16_PARAM)
    tol = dict(g_x=out, g_y=out, g_W=par, g_b=par, g_alpha=par)
    for forward, backward in ((L.forward_fused, L.backward_fused), (L.forward_separable, L.backward_separable)):
        forward()
        for k in tol:
            getattr(L, k).fill_(float("nan"))
        backward()
        torch.cuda.synchronize()
        for k, limit in tol.items():
            e = rel_err(to_np64(getattr(L, k)), ref[k])
            assert e <= limit, f"{backward.__name__} {k}: {e:.3e} > {limit}"


def test_no_event_of_an_earlier_arming():
    """A launch of no stage records nothing, also after an armed call whose events are gone."""
    wl = _wl(3, 64, 40)
    inp = si.make_inputs(wl, seed=1, device="cuda")
    L = GpuLayer(desc_for(wl), inp)
    lib = mhcl.lib()
    lib.mhcl_profile_next_call.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    ev = HipEvents(2)
    assert lib.mhcl_profile_next_call(3, ev.ev[0], ev.ev[1]) == 0
    L.forward_separable()
    L.backward_separable()
    torch.cuda.synchronize()
    kept = L.g_x.clone()
    ev.close()
    L.backward_separable()
    torch.cuda.synchronize()
    assert torch.equal(kept, L.g_x)
