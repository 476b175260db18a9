"""Workspace sizes are answered on the host for every form and operation, also for an empty batch."""
import pytest

import paper_2601_05732_amd as mhcl


@pytest.mark.parametrize("T", [0, 1, 33, 100000])
def test_workspace_sizes(T):
    for io in (mhcl.BF16, mhcl.F32):
        for mode in (mhcl.RES_LITE, mhcl.RES_SK):
            for n in range(1, 6):
                for C in (8, 64, 1000, 1024, 4096):
                    d = mhcl.Desc(n, C, T, io, mode)
                    for op in (mhcl.OP_COEFFS, mhcl.OP_COEFFS_BWD, mhcl.OP_FWD_COEFFS_PRE, mhcl.OP_BWD_FUSED):
                        assert mhcl.workspace_bytes(d, op) >= 256, (n, C, T, io, mode, op)
