"""The Python binding: argument checks, and that what is refused is refused before anything is launched.  Without a GPU every
call ends in a check, and the checks are reached in the order of the arguments; what takes device tensors is marked gpu."""
import ctypes
import gc
import importlib
import os
import shutil
import sys
import types

import numpy as np
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


def calls(m):
    """Every natively marshalled function on small CPU tensors, with the name of its first tensor."""
    z = torch.zeros
    x, bl, a = z(1, 8, 16), z(1, 8, 4), z(16, 4)
    xs, bs = z(2, 16), z(2, 4)
    xm, bm = z(1, 8, 2, 64, dtype=BF16), z(1, 8, 64, dtype=BF16)
    block = m.Block.__new__(m.Block)
    block.c = m.BlockParams(64, 64, 16, 8, 4, 1e-5)
    hid, conv, ssm = z(1, 8, 64, dtype=BF16), z(1, 64, 3, dtype=BF16), z(1, 64, 16)
    return {
        "mamba_conv1d_fwd": ("x", lambda: m.mamba_conv1d_fwd(x, z(16, 4))),
        "mamba_scan_fwd": ("x", lambda: m.mamba_scan_fwd(x, x, a, bl, bl)),
        "mamba_state_step": ("h_out", lambda: m.mamba_state_step(z(2, 16, 4), xs, xs, a, bs, bs)),
        "mamba_conv_state_step": ("h_out", lambda: m.mamba_conv_state_step(z(2, 16, 4), z(2, 16, 3), xs, z(16, 4), None, xs, a, bs, bs)),
        "mamba_state_fork": ("conv_dst", lambda: m.mamba_state_fork(z(1, 2, 16, 3), z(1, 2, 16, 4), z(2, dtype=I32))),
        "mamba_linear_fwd": ("x", lambda: m.mamba_linear_fwd(z(2, 16, dtype=BF16), z(24, 16, dtype=BF16))),
        "mamba_rmsnorm_fwd": ("x", lambda: m.mamba_rmsnorm_fwd(z(2, 16, dtype=BF16), z(16))),
        "mamba_block_fwd": ("hidden", lambda: m.mamba_block_fwd(block, hid)),
        "mamba_block_step": ("hidden", lambda: m.mamba_block_step(block, hid[0, :1], conv, ssm)),
        "mamba_embedding_fwd": ("tokens", lambda: m.mamba_embedding_fwd(z(3, dtype=I32), z(5, 8, dtype=BF16))),
        "mamba_topk_fwd": ("logits", lambda: m.mamba_topk_fwd(z(2, 100, dtype=BF16), 4)),
        "mamba2_ssd_fwd": ("x", lambda: m.mamba2_ssd_fwd(xm, z(1, 8, 2, dtype=BF16), z(2), bm, bm)),
        "mamba2_state_step": ("h_out", lambda: m.mamba2_state_step(z(2, 1, 64, 64), z(2, 1, 64), z(2, 1), z(1), z(2, 64), z(2, 64))),
    }


@pytest.mark.parametrize("name", ["mamba_conv1d_fwd", "mamba_scan_fwd", "mamba_state_step", "mamba_conv_state_step", "mamba_state_fork",
                                  "mamba_linear_fwd", "mamba_rmsnorm_fwd", "mamba_block_fwd", "mamba_block_step", "mamba_embedding_fwd",
                                  "mamba_topk_fwd", "mamba2_ssd_fwd", "mamba2_state_step"])
def test_tensors_not_on_the_gpu_are_refused_by_name(m, name):
    """The first argument of the C function is the first to be named, on a machine without a GPU too: the stream is asked for
    only when all tensors have been checked."""
    first, call = calls(m)[name]
    with pytest.raises(ValueError, match="^%s must live on the GPU$" % first):
        call()


def test_io_type_is_named_as_torch_names_it(m):
    with pytest.raises(TypeError, match=r"^I/O tensors must be float32 or bfloat16, got torch\.float64$"):
        m.mamba_conv1d_fwd(torch.zeros(1, 8, 16, dtype=torch.float64), torch.zeros(16, 4))


@pytest.mark.gpu
def test_wrong_shapes_and_types_are_named_with_what_was_expected(m):
    z = lambda *s, dt=F32: torch.zeros(*s, dtype=dt, device="cuda:0")
    x, w = z(1, 8, 16), z(16, 4)
    for call, error, text in (
            (lambda: m.mamba_conv1d_fwd(x, w, z(15)), ValueError, r"bias must have shape (16,), got (15,)"),
            (lambda: m.mamba_conv1d_fwd(x, w, conv_state_in=z(1, 16)), ValueError, r"conv_state_in must have shape (1, 16, 3), got (1, 16)"),
            (lambda: m.mamba_conv1d_fwd(x, z(16, 4, dt=BF16)), TypeError, r"w must be torch.float32, got torch.bfloat16"),
            (lambda: m.mamba_scan_fwd(x, x, z(16, 4), z(1, 8, 4), z(1, 7, 4)), ValueError, r"Cm must have shape (1, 8, 4), got (1, 7, 4)"),
            (lambda: m.mamba_state_step(z(2, 16, 4), z(2, 16), z(2, 16), z(16, 4), z(2, 4), z(2, 4), parent_idx=z(3, dt=I32)), ValueError,
             r"parent_idx must have shape (2,), got (3,)"),
            (lambda: m.mamba_conv1d_fwd(x.transpose(1, 2), w), ValueError, r"x must be contiguous")):
        with pytest.raises(error) as e:
            call()
        assert str(e.value) == text


def test_numbers_of_other_types_are_taken_as_before(m):
    """eps is whatever float() takes, k any number that is whole where the outputs are given and an integer where they are not."""
    x, logits = torch.zeros(2, 16, dtype=BF16), torch.zeros(2, 100, dtype=BF16)
    idx, val = torch.zeros(2, 8, dtype=I32), torch.zeros(2, 8)
    on_gpu = pytest.raises(ValueError, match="must live on the GPU")          # all other checks of the arguments passed
    for eps in (1e-5, "1e-5", 1, np.float32(1e-5), torch.tensor(1e-5)):
        with on_gpu:
            m.mamba_rmsnorm_fwd(x, torch.zeros(16), eps=eps)
    for k in (8, 8.0, np.int64(8), np.float32(8), torch.tensor(8)):
        with on_gpu:
            m.mamba_topk_fwd(logits, k, idx, val)
    for k in (8, np.int64(8), torch.tensor(8)):
        with on_gpu:
            m.mamba_topk_fwd(logits, k)
    with pytest.raises(TypeError):
        m.mamba_topk_fwd(logits, 8.0)
    with pytest.raises((TypeError, ValueError)):
        m.mamba_topk_fwd(logits, 8.5, idx, val)


@pytest.mark.gpu
def test_fork_takes_parents_and_states_with_further_dimensions(m):
    """Parents as a column (n_out, 1), states with a last dimension of one."""
    conv = torch.randn(2, 3, 16, 3, device="cuda:0")
    ssm = torch.randn(2, 3, 16, 4, device="cuda:0")
    parent = torch.tensor([2, 0, 1, 1, 2], dtype=I32, device="cuda:0")
    want = conv[:, parent.long()], ssm[:, parent.long()]
    for got in (m.mamba_state_fork(conv, ssm, parent), m.mamba_state_fork(conv, ssm, parent[:, None]),
                m.mamba_state_fork(conv[..., None], ssm[..., None], parent)):
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.gpu
def test_linear_returns_every_output_that_is_there(m):
    """An output of no width may be None among the given ones: the others are returned."""
    x = torch.randn(5, 16, device="cuda:0").to(BF16)
    w = torch.randn(24, 16, device="cuda:0").to(BF16)
    a, c = m.mamba_linear_fwd(x, w, splits=[8, 16])
    new = lambda n: torch.empty(5, n, dtype=BF16, device="cuda:0")
    for splits, outs in (([8, 0, 16], [new(8), None, new(16)]), ([0, 8, 16], [None, new(8), new(16)])):
        got = m.mamba_linear_fwd(x, w, splits=splits, outs=outs)
        assert len(got) == 2 and torch.equal(got[0], a) and torch.equal(got[1], c)
    (whole,) = m.mamba_linear_fwd(x, w, splits=[0, 24], outs=[None, new(24)])
    assert torch.equal(whole, torch.cat([a, c], 1))


def test_a_tensor_without_dimensions_is_no_empty_batch(m):
    """What gives the number of rows has to have rows: a scalar is refused, not taken for none of them."""
    z = torch.zeros
    for call in (lambda: m.mamba_state_step(z(2, 16, 4), z(()), z(0, 16), z(16, 4), z(0, 4), z(0, 4)),
                 lambda: m.mamba_conv_state_step(z(2, 16, 4), z(2, 16, 3), z(()), z(16, 4), None, z(0, 16), z(16, 4), z(0, 4), z(0, 4)),
                 lambda: m.mamba2_state_step(z(2, 1, 64, 64), z(()), z(0, 1), z(1), z(0, 64), z(0, 64)),
                 lambda: m.mamba_embedding_fwd(z((), dtype=I32), z(5, 8, dtype=BF16)),
                 lambda: m.mamba_state_fork(z(1, 2, 16, 3), None, z((), dtype=I32))):
        with pytest.raises(ValueError, match="must have at least 1 dimensions, got 0"):
            call()


def test_scan_on_another_stream_allocates_a_workspace_only_where_it_needs_one(m, monkeypatch):
    made = []
    monkeypatch.setattr(m, "_scratch", lambda nbytes, device, stream: made.append(nbytes))
    stream = types.SimpleNamespace(cuda_stream=0)
    for L, D in ((8, 16), (4096, 256)):
        x, bc = torch.zeros(1, L, D), torch.zeros(1, L, 16)
        need = m.mamba_scan_workspace_bytes(1, L, D, 16)
        assert (need > 0) == (L == 4096)
        with pytest.raises(ValueError, match="x must live on the GPU"):
            m.mamba_scan_fwd(x, x, torch.zeros(D, 16), bc, bc, stream=stream)
        assert made == [need] * (need > 0)


def test_a_stream_is_a_stream_whatever_its_truth(m, monkeypatch):
    """Only None stands for the current stream; an object that happens to be false is not one."""
    monkeypatch.setattr(m, "_marshal", types.SimpleNamespace(conv1d_fwd=lambda *a: a[-1]))

    class Empty(types.SimpleNamespace):
        def __len__(self):
            return 0
    assert m.mamba_conv1d_fwd(None, None, stream=Empty(cuda_stream=7)) == 7 and m.mamba_conv1d_fwd(None, None) is None
    with pytest.raises(AttributeError):
        m.mamba_conv1d_fwd(None, None, stream=0)


def test_binding_without_the_marshalling_module_says_how_to_build_it(tmp_path, monkeypatch):
    package = tmp_path / "half_built"
    package.mkdir()
    (package / "__init__.py").write_text("")
    (package / "libmamba_hip.so").write_bytes(b"")
    shutil.copy(os.path.join(ROOT, "paper_2506_01206_amd", "binding.py"), package / "binding.py")
    for name in ("MAMBA_HIP_LIB", "MAMBA_HIP_MARSHAL"):
        monkeypatch.delenv(name, raising=False)
    monkeypatch.syspath_prepend(str(tmp_path))
    with pytest.raises(ImportError, match="python -m paper_2506_01206_amd.build"):
        importlib.import_module("half_built.binding")


@pytest.mark.parametrize("name", ["mamba_conv1d_fwd", "mamba_scan_fwd", "mamba_linear_fwd", "mamba_rmsnorm_fwd", "mamba_topk_fwd", "mamba2_ssd_fwd"])
def test_what_is_no_tensor_or_has_another_rank_is_refused(m, name):
    z, call = torch.zeros, getattr(m, name)
    args = dict(mamba_conv1d_fwd=(z(16, 4),), mamba_scan_fwd=(z(1, 8, 16), z(16, 4), z(1, 8, 4), z(1, 8, 4)), mamba_linear_fwd=(z(24, 16),),
                mamba_rmsnorm_fwd=(z(16),), mamba_topk_fwd=(4,), mamba2_ssd_fwd=(z(1, 8, 2), z(2), z(1, 8, 64), z(1, 8, 64)))[name]
    for no_tensor in (None, 3, "x", [1.0], np.zeros((1, 8, 16), np.float32)):
        with pytest.raises(TypeError, match="must be a tensor"):
            call(no_tensor, *args)
    for shape in ((), (4,), (1, 2, 3, 4, 5)):
        with pytest.raises(ValueError, match="must have . dimensions, got %d" % len(shape)):
            call(z(*shape) if shape else z(()), *args)
    if name == "mamba_scan_fwd":
        for chunk_len in (4.0, "4", None, 1 << 70):
            with pytest.raises((TypeError, OverflowError)):
                call(z(1, 8, 16), *args, chunk_len=chunk_len)


def test_native_entries_take_exactly_their_arguments(m):
    """By position, all of them: one more or one less is an error, and so is a bind without the addresses."""
    counts = dict(conv1d_fwd=9, scan_fwd=16, state_step=14, conv_state_step=21, state_fork=6, linear_fwd=12, rmsnorm_fwd=5, block_fwd=10,
                  block_step=10, embedding_fwd=4, topk_fwd=5, ssd_fwd=15, ssd_step=14)
    assert set(counts) == {n for n in dir(m._marshal) if not n.startswith("_")} - {"bind"}
    for name, n in counts.items():
        for args in ((), (None,) * (n - 1), (None,) * (n + 1)):
            with pytest.raises(TypeError, match="%d arguments expected, got %d" % (n, len(args))):
                getattr(m._marshal, name)(*args)
    for args in ((), (m.MambaError, torch.OutOfMemoryError), (m.MambaError, torch.OutOfMemoryError) + ("no address",) * 16):
        with pytest.raises(TypeError):
            m._marshal.bind(*args)


def test_an_output_that_cannot_be_allocated_raises(m):
    """Errors of torch's allocation come out as torch's own: negative sizes, more memory than there is."""
    x = torch.zeros(1, 8, 16)
    with pytest.raises(RuntimeError):
        m.mamba_conv1d_fwd(x, torch.zeros(16, 0))
    with pytest.raises(RuntimeError):
        m.mamba_topk_fwd(torch.zeros(2, 8, dtype=BF16), 1 << 61)      # (the bytes overflow)


def test_no_references_are_lost_or_kept(m):
    """Outputs that were allocated before a check failed are given back, and the arguments are only borrowed."""
    x, w, y = torch.zeros(1, 8, 16), torch.zeros(16, 4), torch.zeros(1, 8, 16)

    def counts():
        gc.collect()                                     # (exceptions hold the frames that they came through)
        return [sys.getrefcount(o) for o in (x, w, y, None)]
    before = counts()
    for _ in range(200):
        for out, want_state in ((None, True), (y, True), (y, False)):
            with pytest.raises(ValueError):
                m.mamba_conv1d_fwd(x, w, y=out, want_state=want_state)
    del out
    after = counts()
    assert before[:3] == after[:3] and abs(after[3] - before[3]) < 100
