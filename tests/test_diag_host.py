"""diag.layer_stack without layers: empty stacks, no call into the library's kernels."""
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
