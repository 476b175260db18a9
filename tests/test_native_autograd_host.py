"""Host side of the C++ graph nodes (no GPU needed): what they are given and what they refuse."""
import pytest
import torch

from paper_2601_05732_amd import autograd, binding
from paper_2601_05732_amd.autograd import HyperConnection


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
