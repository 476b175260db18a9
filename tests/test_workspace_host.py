"""Workspace sizes are answered on the host, also for an empty batch (what they have to hold:
test_workspace_reuse_host.py), and the shapes the static array takes do not depend on the projection."""
import pytest
import torch

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


def _mfma_slices(n, C, T, M):
    tiles = -(-M // 16)
    kc, tokens = (2 if tiles >= 4 else 4), (128 if tiles <= 3 else 256)
    steps, blocks, ks = n * C // 32, -(-T // tokens), 1
    while ks < 4 and blocks * ks < 256 and steps % (ks * 4 * kc) == 0:
        ks *= 2
    return ks


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
def test_static_array_takes_the_same_shapes_whichever_projection_runs(n):
    """mhcl_fwd_coeffs_pre_static refuses what needs more scratch than its array.  Few tokens take the
    fp64 projection, whose slices are sized differently: the line must lie where the bf16 projection's
    slices and packed W put it (C a multiple of 64), or one slice (any other C, f32 streams)."""
    up = lambda v: -(-v // 256) * 256  # noqa: E731
    for T in (1, 16, 17, 100, 255, 256, 1000, 2227, 4096, 20000, 31000, 31100, 110000):
        for C in (64, 1000, 1024, 2560, 4096, 8192, 20480, 24576, 32768):
            for io in (mhcl.BF16, mhcl.F32):
                for mode in (mhcl.RES_LITE, mhcl.RES_SK):
                    d = mhcl.Desc(n, C, T, io, mode)
                    if io == mhcl.BF16 and C % 64 == 0:
                        ks = _mfma_slices(n, C, T, d.M)
                        want = up(ks * T * d.M * 4) + up(ks * T * 4) + up(n * C // 32 * -(-d.M // 16) * 2048)
                    else:
                        want = up(T * d.M * 4) + up(T * 4)
                    got = mhcl.workspace_bytes(d, mhcl.OP_COEFFS)
                    assert (got > mhcl.STATIC_SCRATCH_BYTES) == (want > mhcl.STATIC_SCRATCH_BYTES), (n, C, T, io, mode)


@pytest.mark.parametrize("n,K", [(8, 96), (8, 112), (8, 128), (6, 128), (5, 110)])
def test_static_array_takes_the_longest_logit_rows_too(n, K):
    """One slice of these fits up to 29000 tokens and more, so split rows of few tokens have to."""
    d = mhcl.Desc(n, 4096, 0, mhcl.F32, mhcl.RES_SUBSET, perm=torch.zeros(K, n, dtype=torch.int8))
    for C in (256, 1000, 4096, 20480):
        d.c.C = C
        for T in list(range(1, 4000, 13)) + list(range(4000, 9000, 5)) + [16 * g + k for g in range(300) for k in (0, 1)][1:]:
            d.c.T = T
            for io in (mhcl.BF16, mhcl.F32) if C % 64 else (mhcl.F32,):
                d.c.io_dtype = io
                assert mhcl.workspace_bytes(d, mhcl.OP_COEFFS) <= mhcl.STATIC_SCRATCH_BYTES, (C, T, io)
