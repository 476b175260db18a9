"""mhcl_coeffs_logits_layers: the bits of one call per layer, whatever number of layers shares a launch, behind each
projection and lane count and at edges of the stage's blocks; and diag.layer_stack over it."""
import pytest
import torch

import paper_2601_05732_amd as mhcl
import synth_inputs as si
from paper_2601_05732_amd import binding, diag
from gpu_harness import desc_for

pytestmark = pytest.mark.gpu

CASES = [(4, 512, 1251, "bf16", "sk", 6), (4, 64, 33, "bf16", "lite", 9), (2, 24, 65, "f32", "sk", 2),
         (5, 128, 1700, "bf16", "sk", 3), (3, 64, 16385, "bf16", "lite", 2), (1, 8, 1, "f32", "lite", 17),
         (4, 1024, 40, "bf16", "sk", 2), (4, 64, 5003, "bf16", "sk", 4), (3, 64, 8192, "bf16", "sk", 2),
         (2, 128, 2700, "bf16", "sk", 7), (1, 64, 4097, "bf16", "sk", 4)]


@pytest.mark.parametrize("room", [1, 2, 8])
@pytest.mark.parametrize("n,C,T,io,mode,L", CASES)
def test_layers_in_shared_launches_give_the_bits_of_single_calls(n, C, T, io, mode, L, room):
    wl = si.Workload("layers", n=n, C=C, T=T, io=io, res_mode=mode, backward=False)
    d = desc_for(wl)
    inp = [si.make_inputs(wl, seed=60 + l, device="cuda") for l in range(L)]
    e = lambda *s: torch.full(s, float("nan"), device="cuda")  # noqa: E731
    H, z, spread = e(L, T, n, n), e(L, T, d.M), e(L, T)
    each = binding.workspace_bytes(d, mhcl.binding.OP_COEFFS_LAYERS)
    assert each > 0
    binding.mhcl_coeffs_logits_layers(d, *[[i[k] for i in inp] for k in ("x", "W", "b", "alpha")], H, z, spread,
                                      torch.empty(room * each, device="cuda", dtype=torch.uint8))
    Hs, zs, ss = diag.layer_stack(wl, L, inp)
    for l in range(L):
        one = [e(T, n, n), e(T, n), e(T, n), e(T, d.M), e(T)]
        binding.mhcl_coeffs_logits(d, *[inp[l][k] for k in ("x", "W", "b", "alpha")], *one,
                                   binding.new_workspace(d, mhcl.OP_COEFFS))
        for joint, stack, single in ((H, Hs, one[0]), (z, zs, one[3]), (spread, ss, one[4])):
            assert torch.equal(joint[l], single) and torch.equal(stack[l], single)


@pytest.mark.parametrize("n,C,T,mode,K", [(5, 64, 70, "lite", 0), (6, 64, 70, "subset", 20), (4, 4096, 4200, "lite", 0)])
def test_forms_whose_layers_do_not_share_launches(n, C, T, mode, K):
    wl = si.Workload("layers", n=n, C=C, T=T, res_mode=mode, n_perm=K, backward=False)
    inp = si.make_inputs(wl, seed=3, device="cuda")
    d = desc_for(wl, perm=inp.get("perm"))
    assert binding.workspace_bytes(d, mhcl.binding.OP_COEFFS_LAYERS) == 0
    e = lambda *s: torch.empty(s, device="cuda")  # noqa: E731
    with pytest.raises(mhcl.MhclError) as err:
        binding.mhcl_coeffs_logits_layers(d, [inp["x"]], [inp["W"]], [inp["b"]], [inp["alpha"]], e(1, T, n, n),
                                          e(1, T, d.M), e(1, T), torch.empty(1 << 20, device="cuda", dtype=torch.uint8))
    assert err.value.status == 2
