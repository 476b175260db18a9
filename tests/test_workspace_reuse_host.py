"""A workspace that is large enough for a batch is large enough for a smaller one: sizes never fall as T
grows, for the backward operations of every form and for the forward wherever the projection's
slices are the fp64 ones (f32 streams, C no multiple of 64, few tokens).  The bf16 projection splits its rows
while its blocks do not fill the chip, into up to sixteen parts as far as the static array holds them and into up to four
anyway, so there the forward's size may fall where the latter split ends; nowhere else.  No size is larger than what some
call of so many tokens or fewer writes."""
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


def _tiles(M):
    return -(-M // 16)


def _few(M):
    """Up to so many tokens the fp64 projection runs where the bf16 one could too."""
    return (2500 if _tiles(M) <= 4 else 5000) // _tiles(M)


def _fullprec_parts(n, C, T, io, M):
    V = 8 if io == mhcl.BF16 else 4
    steps, groups, parts = -(-n * C // (4 * V)), -(-T // 16), 1
    many = steps // 128 * V * _tiles(M) >= (64 if io == mhcl.BF16 else 128)
    while (parts < (32 if groups <= 2 and many else 16) and groups * parts < (448 if _tiles(M) >= 8 else 512)
           and steps >= 16 * parts):
        parts *= 2
    return parts


class _Mfma:
    """The bf16 projection's split of rows."""

    def __init__(self, n, C, M):
        self.K, self.M = n * C, M
        self.kc, self.tok = 2 if _tiles(M) >= 4 else 4, 128 if _tiles(M) <= 3 else 256
        self.steps = self.K // 32
        self.chunks = -(-self.steps // self.kc)
        self.fit = max(0, mhcl.STATIC_SCRATCH_BYTES - self.packed() - 512) // (4 * (M + 1))

    def packed(self):
        return -(-self.steps * _tiles(self.M) * 2048 // 256) * 256

    def small(self, T):   # parts that the workspace has room for whatever the static array holds
        ks = 1
        while ks < 4 and -(-T // self.tok) * ks < 256 and self.steps % (ks * 4 * self.kc) == 0:
            ks *= 2
        return ks

    def parts(self, T):
        blocks = -(-T // self.tok)
        best, best_cost = self.chunks, None
        for p in range(1, min(16, max(self.small(T), self.fit // T)) + 1):
            each = -(-self.chunks // p)
            if p > 1 and (self.chunks < 4 or each < 2 or blocks * p > 768):
                break
            cost = -(-blocks * p // 256) * (each / self.chunks) + blocks * (p / 256 * 4 * self.M / self.K)
            if best_cost is None or cost < 0.9 * best_cost:
                best, best_cost = each, cost
        return -(-self.steps // (best * self.kc))


def _slice_floats(n, C, T, io, M):
    """floats per logit and sum of squares that the projection of the forward writes"""
    if io == mhcl.BF16 and C % 64 == 0 and T > _few(M):
        return _Mfma(n, C, M).parts(T) * T
    p = _fullprec_parts(n, C, T, io, M)
    return T if p == 1 else 2 * p * T


def _reduce_parts(C, T, wide):
    steps = C // 64
    if not wide and -(-T // 128) >= 256:
        return 1
    parts = max(1, min(256 // -(-T // 64), 16, steps))
    return -(-steps // -(-steps // parts))


def test_sizes_hold_what_the_kernels_write():
    """Lower bounds from the shapes: the slices of the projection (in fp64 where the fp64 one splits rows) and of the dot products
    that a call of T tokens writes, the per-token records and vectors of the backward."""
    seen = set()
    for n, mode, K in FORMS:
        for C in (8, 64, 320, 1000, 1024, 1088, 2560, 4096):
            for io in (mhcl.BF16, mhcl.F32):
                for T in (1, 17, 33, 500, 1000, 1250, 1409, 3000, 5003, 8176, 9000, 20000, 40000, 100000):
                    M, (fwd,) = _sizes(n, C, io, mode, K, 20, [T], mhcl.OP_COEFFS)
                    bf16_path = io == mhcl.BF16 and C % 64 == 0
                    packed = bf16_path and T > _few(M)
                    slices = _slice_floats(n, C, T, io, M)
                    seen.add((packed, slices // T))
                    dots, record = n * n + 2 * n, n * n + 2 * n + 1
                    assert fwd >= 4 * slices * (M + 1) + (_Mfma(n, C, M).packed() if packed else 0), (n, mode, C, io, T)
                    _, (bwd,) = _sizes(n, C, io, mode, K, 20, [T], mhcl.OP_COEFFS_BWD)
                    assert bwd >= 4 * (slices * (M + 1) + T * (record + M)), (n, mode, C, io, T)
                    _, (fused,) = _sizes(n, C, io, mode, K, 20, [T], mhcl.OP_BWD_FUSED)
                    wide = n > 4 or mode == mhcl.RES_SUBSET
                    parts = _reduce_parts(C, T, wide) if bf16_path else 1
                    proj = slices if wide or not bf16_path else parts * T
                    assert fused >= 4 * (proj * (M + 1) + T * (parts * dots + record + M)), (n, mode, C, io, T)
    # every kind of split was met: fp64 slices of up to 32 parts, bf16 ones of even and uneven numbers
    assert {(False, 2 * p) for p in (2, 4, 8, 16, 32)} <= seen and {(True, p) for p in (1, 2, 3, 5, 16)} <= seen, seen


@pytest.mark.parametrize("n,mode,K", FORMS)
def test_sizes_hold_no_more_than_some_call_writes(n, mode, K):
    """Upper bounds: the forward's workspace is the slices that a call of T tokens or fewer writes, and packed W; and
    the backward operations have the same slices."""
    for C in (64, 320, 1024, 4096):
        d_M, _ = _sizes(n, C, mhcl.BF16, mode, K, 20, [1], mhcl.OP_COEFFS)
        split, most = _Mfma(n, C, d_M), {}
        use, ends = 0, [64 * k for k in range(1, 1601)]
        for T in ends:
            # (the first token of a block may split into more parts than its last one, up to the array's room)
            first = max((T - 1) // split.tok * split.tok + 1, _few(d_M) + 1)
            if T > _few(d_M):
                use = max(use, split.parts(T) * T, min(split.parts(first) * T, split.fit))
            most[T] = use
        for T in (64, 512, 1024, 1280, 2560, 4096, 5056, 8192, 9344, 16384, 32768, 50048, 102400):
            few = min(T, _few(d_M))
            wide = max([T] + [_slice_floats(n, C, t, mhcl.BF16, d_M) for t in [*range(16, few + 1, 16), few]])
            if wide > T:   # (reserved as if the blocks of tokens times parts were all used up: 4 % more at most)
                wide = int(1.04 * wide)
            slices = max(T, split.small(T) * T, min(most[T], split.fit))
            _, (fwd,) = _sizes(n, C, mhcl.BF16, mode, K, 20, [T], mhcl.OP_COEFFS)
            held = max(4 * slices * (d_M + 1) + split.packed(), 4 * wide * (d_M + 1)) + 1024
            assert fwd <= held, (C, T, fwd, held)
            _, (bwd,) = _sizes(n, C, mhcl.BF16, mode, K, 20, [T], mhcl.OP_COEFFS_BWD)
            rest = 4 * (T * (n * n + 2 * n + 8) + (T + 32) * (16 * _tiles(d_M)) + (T // 32 + 2) * (d_M + 3))
            chunks = max(1, min(256 // -(-n * C // (128 if _tiles(d_M) <= 3 else 64)), -(-T // 256)))
            rest += (4 * chunks * n * C * d_M if chunks > 1 else 0) + split.packed()
            assert bwd <= 4 * max(T, most[T], wide) * (d_M + 1) + rest + 4096, (C, T, bwd)
