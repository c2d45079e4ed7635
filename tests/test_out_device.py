"""An ``out`` that is not on the operands' device is refused before anything is
launched (its address would be handed to the kernels)."""
import pytest
import torch

from paper_cs_9809105_amd import binding as B


class OnGpu(torch.Tensor):
    """A host tensor that says it is on the GPU: only the checks may use it."""
    device = property(lambda self: torch.device("cuda", 0))


def _g(*shape):
    return torch.ones(shape).as_subclass(OnGpu)


def test_new_out():
    dev = torch.device("cuda", 0)
    for out in (torch.ones(3, 4), torch.ones((3, 4), device="meta")):
        with pytest.raises(ValueError, match="device"):
            B._new_out((3, 4), B.HS_F32, dev, out, "out")
    assert B._new_out((3, 4), B.HS_F32, dev, o := _g(3, 4), "out") is o
    with pytest.raises(ValueError, match="device"):
        B._new_out((3, 4), B.HS_F32, torch.device("cuda", 1), _g(3, 4), "out")


def test_entry_points():
    for call in (lambda: B.hs_gemm(_g(3, 5), _g(5, 4), out=torch.ones(3, 4)),
                 lambda: B.hs_gemm_tn(_g(5, 3), _g(5, 4), out=torch.ones(3, 4)),
                 lambda: B.hs_gemm_noalloc(_g(3, 5), _g(5, 4), torch.ones(3, 4)),
                 lambda: B.hs_gemv(_g(3, 5), _g(5), out=torch.ones(3)),
                 lambda: B.hs_nbody(_g(6, 4), out=torch.ones(6, 4))):
        with pytest.raises(ValueError, match="device"):
            call()
