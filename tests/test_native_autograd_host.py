"""Host side of the C++ graph nodes (no GPU needed): what they are given and what they refuse."""
import sys

import pytest
import torch

from paper_2601_05732_amd import autograd, binding
from paper_2601_05732_amd.autograd import HyperConnection, HyperConnectionStack


@pytest.mark.parametrize("table", [torch.arange(5, dtype=torch.int8).repeat(3, 1), torch.arange(7, dtype=torch.int8).repeat(3, 1),
                                   torch.arange(6, dtype=torch.int8), torch.arange(6).repeat(3, 1),
                                   torch.zeros(6, 3, dtype=torch.int8).t()],
                         ids=["narrow", "wide", "one row", "int64", "transposed"])
def test_permutation_tables_that_are_not_k_by_n_int8_are_refused(monkeypatch, table):
    for make in (lambda: binding.Desc(6, 64, 0, res_mode=binding.RES_SUBSET, perm=table),
                 lambda: autograd._native().link(6, 64, 0, binding.BF16, binding.RES_SUBSET, 20, 1e-6, table, 0)):
        with pytest.raises(ValueError, match="perm must be a contiguous int8 tensor"):
            make()
    layer = HyperConnection(6, 64, "subset", device="cpu", perm=torch.arange(6, dtype=torch.int8).repeat(3, 1))
    monkeypatch.setattr(autograd, "_plain", lambda *t: True)
    x = torch.zeros(2, 6, 64)
    assert layer._takes_native(x)
    layer.perm = table                  # (the Python node refuses it)
    assert not layer._takes_native(x)


class _Ends:
    """Stands for the C++ module on the CPU: its ends take only what the kernels can read."""

    def __init__(self, n):
        self.n, self.outs, self.module = n, 0, autograd._native()

    def streams_in(self, x0, link):
        assert x0.is_contiguous() and x0.data_ptr() % 16 == 0
        self.shape = (x0.shape[0], self.n, x0.shape[1])
        self.dtype = x0.dtype
        return x0.unsqueeze(1).expand(-1, self.n, -1).contiguous()

    def readable(self, x, x0, link):
        link = self.module.link(self.n, x0.shape[1], x0.shape[0], binding.F32, binding.RES_SK, 20, 1e-6, None, 0)
        return self.module.readable(x, x0, link)

    def streams_out(self, x, link):
        assert x.shape == self.shape and x.dtype is self.dtype and x.is_contiguous() and x.data_ptr() % 16 == 0 \
            and not x.is_neg()
        self.outs += 1
        return x.sum(dim=1)


class _Copy(HyperConnection):      # a layer that needs no library
    def forward(self, x, f):
        return f(x)


_CHANGES = {"none": lambda x: x, "other type": lambda x: x.double(), "fewer tokens": lambda x: x[:5],
            "other width": lambda x: x[..., :8].contiguous(), "other streams": lambda x: x[:, :2].contiguous(),
            "not contiguous": lambda x: x.transpose(0, 2).contiguous().transpose(0, 2),
            "odd address": lambda x: torch.cat([x.flatten()[:1], x.flatten()])[1:].view_as(x),
            "negated view": torch._neg_view, "subclass": lambda x: x.as_subclass(torch.nn.Buffer)}


@pytest.mark.parametrize("change", _CHANGES)
def test_the_end_of_a_stack_takes_what_the_last_layer_returns(monkeypatch, change):
    n, C, T = 4, 64, 9
    stack = HyperConnectionStack(n, C, [lambda x: x * 2] * 2, device="cpu")
    stack.layers = torch.nn.ModuleList([_Copy(n, C, device="cpu") for _ in range(2)])
    stack.layers[1].register_forward_hook(lambda m, a, x: _CHANGES[change](x))
    ends = _Ends(n)
    monkeypatch.setattr(autograd, "_plain", lambda *ts: all(type(t) is torch.Tensor for t in ts))
    monkeypatch.setattr(autograd, "_native", lambda: ends)
    monkeypatch.setattr(HyperConnection, "_native_link", lambda *a: object())
    x0 = torch.randn(T, C)
    want = _CHANGES[change](x0.unsqueeze(1).expand(-1, n, -1).contiguous() * 4).sum(dim=1)
    assert torch.equal(stack(x0), want)
    assert ends.outs == (change == "none")


@pytest.mark.parametrize("x0", [torch.randn(9, 64).double(), torch._neg_view(torch.randn(9, 64))], ids=["double", "negated view"])
def test_the_start_of_a_stack_copies_in_torch_what_the_kernels_cannot_read(monkeypatch, x0):
    stack = HyperConnectionStack(4, 64, [lambda x: x * 2], device="cpu")
    stack.layers = torch.nn.ModuleList([_Copy(4, 64, device="cpu")])
    monkeypatch.setattr(autograd, "_plain", lambda *t: True)
    monkeypatch.setattr(_Ends, "streams_in", lambda *a: pytest.fail("read by the kernels"))
    ends = _Ends(4)
    monkeypatch.setattr(autograd, "_native", lambda: ends)
    monkeypatch.setattr(HyperConnection, "_native_link", lambda *a: object())
    assert torch.equal(stack(x0), (x0 * 2).unsqueeze(1).expand(-1, 4, -1).sum(dim=1))


def test_a_stack_whose_first_layer_was_wrapped(monkeypatch):
    class Wrapped(torch.nn.Module):
        def __init__(self, inner):
            super().__init__()
            self.inner = inner

        def forward(self, x, f):
            return self.inner(x, f)

    stack = HyperConnectionStack(4, 64, [lambda x: x * 2], device="cpu")
    stack.layers = torch.nn.ModuleList([Wrapped(_Copy(4, 64, device="cpu"))])
    monkeypatch.setattr(autograd, "_plain", lambda *t: True)
    x0 = torch.randn(9, 64)
    assert torch.equal(stack(x0), (x0 * 2).unsqueeze(1).expand(-1, 4, -1).sum(dim=1))


@pytest.mark.parametrize("io", [torch.bfloat16, torch.float32])
def test_the_end_of_a_stack_sums_as_autocast_does(monkeypatch, io):
    stack = HyperConnectionStack(4, 64, [lambda x: x * 2], device="cpu")
    stack.layers = torch.nn.ModuleList([_Copy(4, 64, device="cpu")])
    ends = _Ends(4)
    monkeypatch.setattr(autograd, "_plain", lambda *t: True)
    monkeypatch.setattr(autograd, "_native", lambda: ends)
    monkeypatch.setattr(HyperConnection, "_native_link", lambda *a: object())
    x0 = torch.randn(9, 64).to(io)
    monkeypatch.setattr(torch, "is_autocast_enabled", lambda device=None: device == "cuda")
    stack(x0)
    assert ends.outs == 0                           # left to torch, whose sum autocast turns into one in fp32


def test_without_the_extension_the_python_nodes_are_taken(monkeypatch):
    monkeypatch.setattr(autograd, "_ext", None)
    monkeypatch.delattr("paper_2601_05732_amd._autograd_native", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2601_05732_amd._autograd_native", None)      # its import raises ImportError
    monkeypatch.setattr(autograd, "_plain", lambda *t: True)
    stack = HyperConnectionStack(4, 64, [lambda h: h], device="cpu")
    with pytest.warns(RuntimeWarning, match="graph nodes in C\\+\\+"):
        assert not stack.layers[0]._takes_native(torch.zeros(3, 4, 64))
    assert stack._native_ends(torch.zeros(3, 64)) is None        # (and no second warning)
