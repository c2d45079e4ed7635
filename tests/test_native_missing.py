"""Without its native call path the binding says what to build, as it does
without the library."""
import sys

import pytest

import paper_cs_9809105_amd
from paper_cs_9809105_amd import binding as B


def test_message(monkeypatch):
    import torch
    monkeypatch.setattr(B, "_native_mod", None)
    monkeypatch.delattr(paper_cs_9809105_amd, "_hs_torch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_cs_9809105_amd._hs_torch", None)
    with pytest.raises(RuntimeError, match="_hs_torch.so.*paper_cs_9809105_amd.build"):
        B.hs_gemm(torch.ones(2, 2), torch.ones(2, 2))
