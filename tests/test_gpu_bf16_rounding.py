"""bf16 outputs are rounded by the hardware's conversion: every exponent, sign and upper mantissa with the lower
halves where rounding to nearest even can go wrong (ties, their neighbours, subnormals, overflow, infinities, NaN)."""
import pytest
import torch

import paper_2601_05732_amd as mhcl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("low", [0x0000, 0x0001, 0x7FFF, 0x8000, 0x8001, 0xFFFF])
def test_bf16_outputs_round_to_nearest_even(low):
    T, C = 65536, 8
    gate = ((torch.arange(T, dtype=torch.int64) << 16) + low).to(torch.int32).view(torch.float32).reshape(T, 1)
    d = mhcl.Desc(1, C, T, mhcl.BF16, mhcl.RES_LITE)
    x = torch.ones(T, 1, C, device="cuda", dtype=torch.bfloat16)
    h = torch.empty(T, C, device="cuda", dtype=torch.bfloat16)
    mhcl.mhcl_pre(d, x, gate.cuda(), h)            # h = gate * 1, rounded once
    want = (gate + 0.0).to(torch.bfloat16).expand(T, C)    # on the host; the sum starts at +0, so -0 becomes +0
    h = h.cpu()
    nan = gate.isnan().expand(T, C)
    assert torch.equal(h.isnan(), nan)
    assert torch.equal(h.view(torch.int16)[~nan], want.contiguous().view(torch.int16)[~nan])
