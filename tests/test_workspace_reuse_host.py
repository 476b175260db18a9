"""A workspace that is large enough for a batch is large enough for a smaller one: sizes never fall as T
grows, for the backward operations of every form and for the forward wherever the projection's
slices are the fp64 ones (f32 streams, C no multiple of 64, few tokens).  The bf16 projection splits its rows
up to four ways while its blocks do not fill the chip, so there the forward's size may fall where a
split ends; nowhere else."""
import ctypes
import random

import pytest
import torch

import paper_2601_05732_amd as mhcl

FORMS = [(n, mode, 0) for mode in (mhcl.RES_LITE, mhcl.RES_SK) for n in range(1, 6)]
FORMS += [(n, mhcl.RES_SUBSET, K) for n, K in ((1, 1), (2, 20), (4, 50), (5, 64), (8, 64), (8, 111), (6, 128))]


def _sizes(n, C, io, mode, K, iters, tokens, op):
    perm = torch.zeros(K, n, dtype=torch.int8) if K else None
    d = mhcl.Desc(n, C, 0, io, mode, iters, perm=perm)
    out = []
    for T in tokens:
        d.c.T = T
        out.append(mhcl.lib().mhcl_workspace_bytes(ctypes.byref(d.c), op))
        assert out[-1] >= 256
    return d.M, out


def _tokens(seed):
    rng = random.Random(seed)
    edges = [e + k for e in (256, 500, 512, 555, 833, 1024, 1250, 2048, 2500, 4096, 8176, 8192, 11250, 16384, 23750,
                             32640, 32768, 49152, 65536, 131072, 200000) for k in (-65, -16, -1, 0, 1, 16, 64)]
    return sorted(set([1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 128, 129] + edges
                      + [int(2 ** rng.uniform(0, 18)) for _ in range(60)]))


def _never_falls(tokens, sizes, what):
    for i in range(1, len(tokens)):
        assert sizes[i] >= sizes[i - 1], (what, tokens[i - 1], sizes[i - 1], tokens[i], sizes[i])


@pytest.mark.parametrize("n,mode,K", FORMS)
def test_sizes_of_the_backward_never_fall(n, mode, K):
    tokens = _tokens(n)
    for C in (8, 40, 64, 320, 768, 1000, 1024, 2560, 4096):
        for io in (mhcl.BF16, mhcl.F32):
            for iters in (1, 32) if mode == mhcl.RES_SK else (20,):
                for op in (mhcl.OP_COEFFS_BWD, mhcl.OP_BWD_FUSED):
                    _never_falls(tokens, _sizes(n, C, io, mode, K, iters, tokens, op)[1], (C, io, iters, op))


@pytest.mark.parametrize("n,mode,K", FORMS)
def test_sizes_of_the_forward(n, mode, K):
    tokens = _tokens(n + 10)
    for C in (8, 40, 64, 320, 768, 1000, 1024, 2560, 4096):
        for io in (mhcl.BF16, mhcl.F32):
            for op in (mhcl.OP_COEFFS, mhcl.OP_FWD_COEFFS_PRE):
                M, sizes = _sizes(n, C, io, mode, K, 20, tokens, op)
                if io == mhcl.F32 or C % 64:
                    _never_falls(tokens, sizes, (C, io, op))
                    continue
                # the slices of the bf16 projection alone, at every T
                tiles = -(-M // 16)
                block, kc, steps = (128, 4, n * C // 32) if tiles <= 3 else (256, 2 if tiles >= 4 else 4, n * C // 32)

                def slices(T):
                    ks = 1
                    while ks < 4 and -(-T // block) * ks < 256 and steps % (ks * 4 * kc) == 0:
                        ks *= 2
                    return ks * T

                for i in range(1, len(tokens)):
                    if slices(tokens[i - 1]) <= slices(tokens[i]):
                        assert sizes[i] >= sizes[i - 1], (C, io, op, tokens[i - 1], tokens[i])


def _fullprec_parts(n, C, T, io):
    V = 8 if io == mhcl.BF16 else 4
    steps, groups, parts = -(-n * C // (4 * V)), -(-T // 16), 1
    while parts < 16 and groups * parts < 512 and steps >= 16 * parts:
        parts *= 2
    return parts


def _reduce_parts(C, T, wide):
    steps = C // 64
    if not wide and -(-T // 128) >= 256:
        return 1
    parts = max(1, min(256 // -(-T // 64), 16, steps))
    return -(-steps // -(-steps // parts))


def test_sizes_hold_what_the_kernels_write():
    """Lower bounds from the shapes: the slices of the projection and of the dot products that a call of
    T tokens writes, the per-token records and vectors of the backward."""
    for n, mode, K in FORMS:
        for C in (8, 64, 1000, 1024, 1088, 4096):
            for io in (mhcl.BF16, mhcl.F32):
                for T in (1, 33, 500, 1000, 1250, 8176, 20000, 100000):
                    M, (fwd,) = _sizes(n, C, io, mode, K, 20, [T], mhcl.OP_COEFFS)
                    tiles = -(-M // 16)
                    bf16_path = io == mhcl.BF16 and C % 64 == 0
                    few = not bf16_path or T * tiles <= (2500 if tiles <= 4 else 5000)
                    slices = _fullprec_parts(n, C, T, io) if few else 1
                    dots, record = n * n + 2 * n, n * n + 2 * n + 1
                    assert fwd >= 4 * slices * T * (M + 1)
                    _, (bwd,) = _sizes(n, C, io, mode, K, 20, [T], mhcl.OP_COEFFS_BWD)
                    assert bwd >= 4 * T * (slices * (M + 1) + record + M)
                    _, (fused,) = _sizes(n, C, io, mode, K, 20, [T], mhcl.OP_BWD_FUSED)
                    wide = n > 4 or mode == mhcl.RES_SUBSET
                    parts = _reduce_parts(C, T, wide) if bf16_path else 1
                    proj = slices if wide or not bf16_path else parts
                    assert fused >= 4 * T * (proj * (M + 1) + parts * dots + record + M), (n, mode, C, io, T)
