"""The Python binding: argument checks, and that what is refused is refused before anything is launched.  Without a GPU every
call ends in a check, and the checks are reached in the order of the arguments; what takes device tensors is marked gpu."""
import ctypes
import os
import types

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BF16, F32, I32 = torch.bfloat16, torch.float32, torch.int32


@pytest.fixture(scope="module")
def m():
    if not os.path.exists(os.path.join(ROOT, "paper_2506_01206_amd", "libmamba_hip.so")):
        from paper_2506_01206_amd import build
        build.build()
    from paper_2506_01206_amd import binding
    return binding


def test_linear_refuses_negative_output_widths(m):
    """A width below zero is not the same as no further output: the remaining widths no longer add up to the rows of w."""
    x, w = torch.zeros(2, 16, dtype=BF16), torch.zeros(24, 16, dtype=BF16)
    for splits in ([32, -8], [-8, 32], [40, -8, -8], [24, 8, -8], [32, -1, -7]):
        with pytest.raises(RuntimeError, match="negative dimension"):
            m.mamba_linear_fwd(x, w, splits=splits)


def test_block_parameters_are_read_at_each_call(m, monkeypatch):
    """What goes to the library is the parameter structure a block holds now: nothing keeps the address of an earlier one."""
    monkeypatch.setattr(m, "_marshal", types.SimpleNamespace(block_fwd=lambda address, *a: address, block_step=lambda address, *a: address))
    block = m.Block.__new__(m.Block)
    for d_inner in (64, 128):
        block.c = m.BlockParams(64, d_inner, 16, 8, 4, 1e-5)
        assert m.mamba_block_fwd(block, None) == m.mamba_block_step(block, None, None, None) == ctypes.addressof(block.c)
