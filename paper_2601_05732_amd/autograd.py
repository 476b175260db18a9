"""`torch.autograd` front end of the hyper-connection layer (paper Sec. 2 Eq. 1,
Sec. 3.2) and a stack of such layers around caller-supplied layer functions.

Every tensor operation of the layer runs in ``libmhcl.so``; this module only
wires the library calls into autograd's graph.  One layer is

    h     = H_pre x                  (mhcl_fwd_coeffs_pre: coefficients + h)
    y     = f(h)                     (the caller's function, ordinary autograd)
    x_out = H_res x + H_post^T y     (mhcl_post)

and its backward, once the gradient on x_out has arrived, is

    g_y                    = sum_i H_post[i] g_xout[i]   (the pre-aggregate kernel run on g_xout)
    g_h                    = backward of f               (autograd)
    g_x, g_W, g_b, g_alpha = mhcl_bwd_fused(x, y, g_xout, g_h)

The graph nodes of plain calls are C++ (``torch_ext/autograd.cpp``: the same calls and gradients at a third of the
host time); calls under function transforms, tracing or dispatch modes, with tensor subclasses, or that an argument
check will refuse, or where the extension is missing, take the nodes below.

The two graph nodes of a layer share a small link object: the node of the post
update hands g_xout and y over to the node of the coefficients, whose backward
runs the fused kernel and returns the whole g_x.  Autograd runs the post node
first because h reaches x_out only through y.

Initialisation follows Sec. 4 ("Initialization"): W = 0, alpha = 0.01,
b_res = -8 except 0 for the identity permutation (or the diagonal in the
Sinkhorn-Knopp form), b_pre = b_post = -1 except +1 for one stream.

The paper does not define how the n streams are created at the network's input
and merged at its output; :class:`HyperConnectionStack` replicates the input
into every stream and sums the streams at the end (a choice, not the paper's).
"""
from __future__ import annotations

import math
import warnings

import torch

from . import binding as mhcl
from .layer import PHASE_G_X, PHASE_G_XOUT, PHASE_X, empty_stream


_ext = None


def _native():
    """The C++ graph nodes, or None, after a warning, where the extension is missing or was built for another torch or
    Python: the nodes below make the same calls into the library (which itself has no replacement: without it this raises)."""
    global _ext
    if _ext is None:
        mhcl.lib()
        try:
            from . import _autograd_native
            _ext = _autograd_native
        except ImportError as e:
            warnings.warn(f"the graph nodes in C++ cannot be loaded ({e}): those in Python take two to three times the host "
                          "time; `python -m paper_2601_05732_amd.build` builds them", RuntimeWarning, stacklevel=2)
            _ext = False
    return _ext or None


def _plain(*tensors) -> bool:
    """Whether nothing but plain autograd looks at a call on these GPU tensors: no subclass, function transform,
    forward-mode level, dispatch or function mode, trace or compilation (the C++ nodes know none of them).
    A default device (torch.set_default_device, `with torch.device(...)`) is a function mode as well."""
    try:
        C = torch._C
        return (all(type(t) in (torch.Tensor, torch.nn.Parameter) and t.is_cuda for t in tensors)
                and not C._are_functorch_transforms_active() and C._len_torch_dispatch_stack() == 0
                and C._len_torch_function_stack() == 0 and C._get_tracing_state() is None
                and torch.autograd.forward_ad._current_level < 0 and not torch.compiler.is_compiling())
    except AttributeError:      # a torch without one of these
        return False


_IO = {torch.bfloat16: mhcl.BF16, torch.float32: mhcl.F32}


class _Link:
    """What the post node leaves for the coefficient node of the same layer."""
    __slots__ = ("y", "g_xout", "H_pre", "g_x_phase", "perm")

    def __init__(self, g_x_phase=PHASE_G_X, perm=None):
        self.y = self.g_xout = self.H_pre = None
        self.g_x_phase = g_x_phase
        self.perm = perm      # int8 [K, n] table of the permutation-subset form, else None


def _desc(x, res_mode, sk_iters, eps, perm=None):
    T, n, C = x.shape
    io = _IO[x.dtype]
    return mhcl.Desc(n, C, T, io, res_mode, sk_iters, eps, perm)


class _CoeffsPre(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, W, b, alpha, link, res_mode, sk_iters, eps):
        d = _desc(x, res_mode, sk_iters, eps, link.perm)
        T, n, C = x.shape
        f = torch.float32
        H_res = torch.empty(T, n, n, device=x.device, dtype=f)
        H_pre = torch.empty(T, n, device=x.device, dtype=f)
        H_post = torch.empty(T, n, device=x.device, dtype=f)
        h = torch.empty(T, C, device=x.device, dtype=x.dtype)
        ws = mhcl.new_workspace(d, mhcl.OP_FWD_COEFFS_PRE, x.device)
        mhcl.mhcl_fwd_coeffs_pre(d, x, W, b, alpha, H_res, H_pre, H_post, h, ws)
        ctx.save_for_backward(x, W, b, alpha)
        ctx.link, ctx.d = link, d
        link.H_pre = H_pre
        ctx.mark_non_differentiable(H_pre)
        ctx.set_materialize_grads(False)     # the gradients on H_* are not read: no zeros for them
        return h, H_res, H_post, H_pre

    @staticmethod
    def backward(ctx, g_h, _g_H_res, _g_H_post, _g_H_pre):
        x, W, b, alpha = ctx.saved_tensors
        d, link = ctx.d, ctx.link
        T, n, C = x.shape
        if link.y is None:
            raise RuntimeError("hyper-connection backward: the post update of this layer was never run")
        g_xout = link.g_xout if link.g_xout is not None else torch.zeros_like(x)
        g_h = torch.zeros(T, C, device=x.device, dtype=x.dtype) if g_h is None else g_h.contiguous()
        f = torch.float32
        g_x = empty_stream(x.shape, x.dtype, x.device, link.g_x_phase)
        g_W, g_b = torch.empty_like(W, dtype=f), torch.empty_like(b, dtype=f)
        g_alpha = torch.empty(3, device=x.device, dtype=f)
        ws = mhcl.new_workspace(d, mhcl.OP_BWD_FUSED, x.device)
        # g_y went out through the post node already: not asked for again
        mhcl.mhcl_bwd_fused(d, x, link.y, W, b, alpha, g_xout, g_h, g_x, None, g_W, g_b, g_alpha, ws)
        link.y = link.g_xout = None
        return g_x, g_W, g_b, g_alpha, None, None, None, None


class _Post(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, y, H_res, H_post, link, res_mode, sk_iters, eps):
        d = _desc(x, res_mode, sk_iters, eps, link.perm)
        y = y.contiguous()
        x_out = empty_stream(x.shape, x.dtype, x.device, PHASE_X)
        mhcl.mhcl_post(d, x, y, H_res, H_post, x_out)
        ctx.save_for_backward(H_res, H_post)
        ctx.link, ctx.d = link, d
        link.y = y
        return x_out

    @staticmethod
    def backward(ctx, g_xout):
        H_res, H_post = ctx.saved_tensors
        d, link = ctx.d, ctx.link
        g_xout = g_xout.contiguous()
        link.g_xout = g_xout
        g_y = torch.empty(d.T, d.C, device=g_xout.device, dtype=g_xout.dtype)
        mhcl.mhcl_pre(d, g_xout, H_post, g_y)            # g_y = sum_i H_post[i] g_xout[i]
        # x and the coefficients get their gradients from the coefficient node (fused kernel), which
        # autograd runs once this node is done, also where no gradient reaches it through f
        return None, g_y, None, None, None, None, None, None


def init_params(n: int, C: int, res_mode: int = mhcl.RES_LITE, one_index: int = 0, device="cuda",
                n_perm: int = 0):
    """W, b, alpha at the paper's initialisation (Sec. 4, "Initialization").  For a permutation
    subset (``n_perm`` rows) the identity is expected as the table's first row."""
    R = {mhcl.RES_LITE: math.factorial(n), mhcl.RES_SK: n * n, mhcl.RES_SUBSET: n_perm}[res_mode]
    b = torch.full((R + 2 * n,), -1.0, dtype=torch.float32)
    b[:R] = -8.0
    if res_mode in (mhcl.RES_LITE, mhcl.RES_SUBSET):
        b[0] = 0.0                         # the identity: first in lexicographic order / first row of the table
    else:
        b[:R:n + 1] = 0.0                  # the diagonal
    b[R + one_index] = 1.0
    b[R + n + one_index] = 1.0
    W = torch.zeros(n * C, R + 2 * n, dtype=torch.float32)
    alpha = torch.full((3,), 0.01, dtype=torch.float32)
    return W.to(device), b.to(device), alpha.to(device)


class HyperConnection(torch.nn.Module):
    """One layer: ``x_out = H_res x + H_post^T f(H_pre x)`` on ``x [T, n, C]``."""

    def __init__(self, n: int, C: int, res_mode: str = "lite", sk_iters: int = 20, eps: float = 1e-6,
                 one_index: int = 0, device="cuda", layer_index: int = 0, perm=None):
        """res_mode: "lite" (all n! permutations), "sk" (Sinkhorn-Knopp) or "subset" (Sec. 5: only
        the K permutations in ``perm``, an int8 tensor [K, n] with the identity as its first row,
        n up to 8)."""
        super().__init__()
        self.n, self.C = n, C
        if (res_mode == "subset") != (perm is not None):
            raise ValueError("perm goes with res_mode 'subset', and only with it")
        # g_x of this layer is g_xout of the one below: alternate the two gradient phases
        # so that x, g_xout and g_x of a layer all differ (see layer.empty_stream)
        self.g_x_phase = PHASE_G_X if layer_index % 2 == 0 else PHASE_G_XOUT
        self.res_mode = {"lite": mhcl.RES_LITE, "sk": mhcl.RES_SK, "subset": mhcl.RES_SUBSET}[res_mode]
        self.sk_iters, self.eps = sk_iters, eps
        if perm is not None:
            self.register_buffer("perm", perm.to(device=device, dtype=torch.int8).contiguous())
        else:
            self.perm = None
        W, b, alpha = init_params(n, C, self.res_mode, one_index, device,
                                  n_perm=0 if perm is None else int(perm.shape[0]))
        self.W, self.b, self.alpha = (torch.nn.Parameter(t) for t in (W, b, alpha))

    def _takes_native(self, x) -> bool:
        W, b, alpha, perm, f = self.W, self.b, self.alpha, self.perm, torch.float32
        if x.dtype not in _IO or not _plain(x, W, b, alpha, *(() if perm is None else (perm,))) or _native() is None:
            return False
        if perm is not None and not (perm.dtype is torch.int8 and perm.dim() == 2 and perm.shape[1] == self.n
                                     and perm.is_contiguous()):
            return False
        R = {mhcl.RES_LITE: math.factorial(self.n), mhcl.RES_SK: self.n * self.n,
             mhcl.RES_SUBSET: 0 if perm is None else perm.shape[0]}[self.res_mode]
        M = R + 2 * self.n
        return (W.dtype is f and b.dtype is f and alpha.dtype is f and W.shape == (self.n * self.C, M) and b.shape == (M,)
                and alpha.shape == (3,) and W.is_contiguous() and b.is_contiguous() and alpha.is_contiguous())

    def _native_link(self, x, g_x_phase):
        return _native().link(self.n, self.C, x.shape[0], _IO[x.dtype], self.res_mode, self.sk_iters, self.eps, self.perm,
                              g_x_phase)

    def forward(self, x: torch.Tensor, f):
        if x.dim() != 3 or x.shape[1] != self.n or x.shape[2] != self.C:
            raise ValueError(f"x must be [T, {self.n}, {self.C}], got {tuple(x.shape)}")
        x = x.contiguous()
        if self._takes_native(x):
            nodes, T = _native(), x.shape[0]
            link = self._native_link(x, self.g_x_phase)
            h, H_res, H_post = nodes.coeffs_pre(x, self.W, self.b, self.alpha, link)
            y = f(h)
            if not (isinstance(y, torch.Tensor) and y.is_cuda and y.dtype is x.dtype and y.shape == (T, self.C)):
                mhcl._ptr(y.contiguous(), x.dtype, (T, self.C), "y")      # raises
            return nodes.post(x, y, H_res, H_post, link)
        link = _Link(self.g_x_phase, self.perm)
        cfg = (self.res_mode, self.sk_iters, self.eps)
        h, H_res, H_post, _ = _CoeffsPre.apply(x, self.W, self.b, self.alpha, link, *cfg)
        y = f(h)
        return _Post.apply(x, y, H_res, H_post, link, *cfg)


def _dense(t: torch.Tensor) -> torch.Tensor:
    """`t` contiguous and 16-byte aligned, as the kernels read it."""
    t = t.contiguous()
    return t if t.data_ptr() % 16 == 0 else t.clone()


class HyperConnectionStack(torch.nn.Module):
    """``len(fs)`` layers around the callables ``fs``.  Input ``[T, C]`` is
    copied into the n streams, the output is the sum of the streams: the paper
    leaves both ends open, this is one choice."""

    def __init__(self, n: int, C: int, fs, res_mode: str = "lite", device="cuda", **kw):
        super().__init__()
        self.n = n
        self.fs = list(fs)
        self.mods = torch.nn.ModuleList([f for f in self.fs if isinstance(f, torch.nn.Module)])
        self.layers = torch.nn.ModuleList(
            [HyperConnection(n, C, res_mode, one_index=l % n, device=device, layer_index=l, **kw)
             for l in range(len(self.fs))])

    def _native_ends(self, x0):
        """What the kernels of the ends share, or None where they cannot read x0 (then torch copies and sums)."""
        first = self.layers[0] if len(self.layers) else None
        if not (isinstance(first, HyperConnection) and first.n == self.n and _plain(x0) and x0.dtype in _IO and x0.dim() == 2
                and x0.shape[1] == first.C and not x0.is_neg() and _native() is not None):
            return None
        # (the gradient on the last layer's x_out lies as a further layer's g_x would)
        return first._native_link(x0, PHASE_G_X if len(self.layers) % 2 == 0 else PHASE_G_XOUT)

    def forward(self, x0: torch.Tensor):
        ends = self._native_ends(x0)
        x = x0.unsqueeze(1).expand(-1, self.n, -1).contiguous() if ends is None else _native().streams_in(_dense(x0), ends)
        for layer, f in zip(self.layers, self.fs):
            x = layer(x, f)
        # (a layer is a module: hooks, or what it was replaced with, may return another tensor than the layer's own; under
        # autocast torch's sum is in fp32 and returns fp32)
        if (ends is None or type(x) is not torch.Tensor or not _native().readable(x, x0, ends)
                or torch.is_autocast_enabled("cuda")):
            return x.sum(dim=1)
        return _native().streams_out(x, ends)
