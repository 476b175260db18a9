"""diag.layer_stack without layers: empty stacks, no call into the library's kernels; and how often it draws its inputs."""
import pytest
import torch

import synth_inputs as si
from paper_2601_05732_amd import diag


@pytest.mark.parametrize("T", [0, 3, 8])
def test_no_layers(T):
    wl = si.Workload("none", n=3, C=64, T=T, res_mode="sk")
    H, z, spread = diag.layer_stack(wl, 0, [], device="cpu")
    assert H.shape == (0, T, 3, 3) and z.shape == (0, T, wl.M) and spread.shape == (0, T)
    assert H.dtype == z.dtype == spread.dtype == torch.float32


class _Drawn:
    """A sequence that makes an item whenever it is asked for one."""

    def __init__(self):
        self.asked = []

    def __getitem__(self, l):
        self.asked.append(l)
        return dict(x=l, W=l, b=l, alpha=l)


def test_a_sequence_that_draws_its_items_is_asked_once_for_each(monkeypatch):
    wl = si.Workload("drawn", n=4, C=64, T=8, res_mode="sk")
    seen, inputs = [], _Drawn()
    monkeypatch.setattr(diag.mhcl, "mhcl_coeffs_logits_layers", lambda *a: pytest.fail("all layers at once"))
    monkeypatch.setattr(diag.mhcl, "mhcl_coeffs_logits", lambda d, *a: seen.append(a[:4]))
    diag.layer_stack(wl, 3, inputs, device="cpu")
    assert inputs.asked == [0, 1, 2] and seen == [(l,) * 4 for l in range(3)]
