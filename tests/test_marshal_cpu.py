"""The native marshalling refuses what the Python one did, with the same kinds of errors, before anything reaches a device."""
import pytest
import torch

from paper_2512_12131_amd import binding as B
from paper_2512_12131_amd import build

X, WD, WU = torch.zeros(4, 16), torch.zeros(8, 16), torch.zeros(24, 8)
WIDE = torch.zeros(4, 48)[:, :16]      # rows 48 apart


@pytest.mark.parametrize("error,call", [
    (ValueError, lambda: B.lr_linear_fwd(X[0], WD, WU)),                          # not two dimensions
    (ValueError, lambda: B.lr_group_fwd(X, None, 1e-5, B.LR_NORM_NONE, WD, WU)),  # weights of members are stacked
    (B.LrError, lambda: B.lr_linear_fwd(X.double(), WD, WU)),                     # a type that the library does not take
    (B.LrError, lambda: B.lr_attention_gqa_fwd(X.half(), X.half(), X.half(), 1, 4, 1, 1, 16)),
    (AssertionError, lambda: B.lr_linear_fwd(torch.zeros(16, 4).t(), WD, WU)),    # rows that are not contiguous
    (AssertionError, lambda: B.lr_linear_fwd_static(X, WD, WU, torch.zeros(4, 8), torch.zeros(4, 23))),
    (AssertionError, lambda: B.lr_attention_gqa_bwd(X, X, torch.zeros(4, 32)[:, :16], X, X, X, 1, 4, 1, 1, 16)),
    (TypeError, lambda: B.lr_swiglu_fwd(X, 1.0)),
    (TypeError, lambda: B.lr_linear_fwd(X, WD, WU, act="silu")),
])
def test_refused(error, call):
    with pytest.raises(error):
        call()


# One row stride is passed for these operands: rows of any other distance would be read, or written, at wrong places.
@pytest.mark.parametrize("call", [
    lambda: B.lr_attention_fwd(X, WIDE, X, 1, 4, 1, 16), lambda: B.lr_attention_fwd(X, X, WIDE, 1, 4, 1, 16),
    lambda: B.lr_attention_bwd(X, X, X, WIDE, X, X, 1, 4, 1, 16), lambda: B.lr_attention_bwd(X, X, X, X, WIDE, X, 1, 4, 1, 16),
    lambda: B.lr_attention_gqa_fwd(X, X, WIDE, 1, 4, 1, 1, 16),
    lambda: B.lr_attention_gqa_bwd(WIDE, X, X, X, WIDE, X, 1, 4, 1, 1, 16), lambda: B.lr_attention_gqa_bwd(WIDE, X, X, WIDE, X, X, 1, 4, 1, 1, 16),
    lambda: B.lr_swiglu_fwd(WIDE, X), lambda: B.lr_swiglu_bwd(X, WIDE, X), lambda: B.lr_swiglu_bwd(WIDE, WIDE, X),
])
def test_operands_of_one_row_stride(call):
    with pytest.raises(AssertionError):
        call()


# ... but dense memory of as many elements is the same rows whatever its shape.
@pytest.mark.skipif(torch.cuda.is_available(), reason="goes on to a device that is not there")
@pytest.mark.parametrize("call", [
    lambda: B.lr_attention_bwd(X, X.view(2, 2, 16), X.view(8, 8), X.view(2, 2, 1, 16), X.view(-1), X, 1, 4, 1, 16),
    lambda: B.lr_attention_gqa_bwd(X, X, X, X.view(2, 2, 1, 16), X.view(8, 8), X, 1, 4, 1, 1, 16),
    lambda: B.lr_swiglu_fwd(X, X.view(2, 2, 16)), lambda: B.lr_swiglu_bwd(X, X.view(64), X.view(2, 2, 16)),
    lambda: B.lr_swiglu_fwd(WIDE[:1], X[:1].view(1, 1, 16)),
])
def test_dense_operands_of_other_shapes(call):
    with pytest.raises((RuntimeError, B.LrError)):      # (not an AssertionError)
        call()


@pytest.mark.parametrize("call", [
    lambda: B.lr_attention_bwd(X, X, X, X.view(2, 2, 16)[:, :, :8], X, X, 1, 4, 1, 16), lambda: B.lr_swiglu_fwd(X, torch.zeros(4, 32)),
    lambda: B.lr_swiglu_fwd(X, torch.zeros(2, 4, 16)), lambda: B.lr_swiglu_fwd(WIDE, X.view(2, 2, 16)),
    lambda: B.lr_attention_fwd(X, X, X.t().contiguous().t(), 1, 4, 1, 16),
    lambda: B.lr_attention_gqa_fwd(X, X, X.view(2, 2, 16), 1, 4, 1, 1, 16), lambda: B.lr_attention_gqa_bwd(X, X, X.view(2, 2, 16), X, X, X, 1, 4, 1, 1, 16),
    lambda: B.lr_attention_gqa_fwd(X[:1], X[:1], WIDE[:1], 1, 1, 1, 1, 16),
])
def test_other_shapes_of_other_memory(call):
    with pytest.raises(AssertionError):
        call()


# No stride is passed for these: of anything but dense memory other elements would be read or written, of a broadcast tensor (the
# gradient of a sum, say) elements past its end.
ONE, G2 = torch.zeros(()), torch.zeros(2, 24, 8)
DY, DESC = ONE.expand(2, 4, 24), B.make_block_desc(1, 4, 128, 1, 128, 256, 256, 32)
Z, Z2, GAMMA, STAT, T128 = torch.zeros(4, 8), torch.zeros(4, 16), torch.zeros(16), torch.zeros(4), torch.zeros(4, 128)
PARAMS = {n: torch.zeros(8) for n in B.PARAM_NAMES}
CKPT, SAVED = ({n: torch.zeros(8) for n, _ in c._fields_} for c in (B.BlockCkpt, B.BlockSaved))


@pytest.mark.parametrize("call", [
    lambda: B.lr_linear_fwd(X, WD.t().contiguous().t(), WU), lambda: B.lr_linear_fwd(X, WD, ONE.expand(24, 8)),
    lambda: B.lr_linear_bwd(X, WD, WU, Z2[:, :8], torch.zeros(4, 24)),
    lambda: B.lr_linear_bwd(X, WD, WU, Z, torch.zeros(4, 24), grads=(torch.zeros(8, 32)[:, :16], WU)),
    lambda: B.lr_group_fwd(X, ONE.expand(16), 1e-5, B.LR_NORM_ONLINE, torch.zeros(16, 16), G2),
    lambda: B.lr_group_bwd(X, None, 1e-5, B.LR_NORM_NONE, torch.zeros(16, 16), G2, Z2, None, DY),
    lambda: B.lr_group_bwd(X, None, 1e-5, B.LR_NORM_NONE, torch.zeros(16, 16), G2, Z2, None, DY.contiguous(), grads=(None, X, G2.transpose(1, 2))),
    lambda: B.lr_attention_gqa_bwd(X, X, X, X, X, ONE.expand(1, 1, 4), 1, 4, 1, 1, 16),
    lambda: B.lr_attention_bwd(X, X, X, X, X, ONE.expand(1, 1, 4), 1, 4, 1, 16),
    lambda: B.lr_rmsnorm_apply(X, GAMMA, ONE.expand(4), 1e-5), lambda: B.lr_rmsnorm_bwd(X, ONE.expand(16), STAT, 1e-5, X),
    lambda: B.lr_block_fwd(DESC, PARAMS, ONE.expand(4, 128)), lambda: B.lr_block_bwd(DESC, PARAMS, T128, ONE.expand(4, 128), CKPT),
    lambda: B.lr_block_bwd_saved(DESC, PARAMS, T128, ONE.expand(4, 128), CKPT, SAVED),
    lambda: B.lr_block_lax_bwd(DESC, PARAMS, T128, ONE.expand(4, 128), CKPT), lambda: B.lr_block_lax_fwd(DESC, PARAMS, ONE.expand(4, 128)),
    lambda: B.lr_block_fwd_save(DESC, PARAMS, ONE.expand(4, 128)), lambda: B.lr_block_fwd(DESC, {**PARAMS, "w_up_d": G2[:, :, 0]}, T128),
    lambda: B.make_block_desc(1, 4, 128, 1, 128, 256, 256, 32, rope=(torch.zeros(4, 128)[:, :64], torch.zeros(4, 64))),
])
def test_operands_without_a_stride_are_dense(call):
    with pytest.raises(AssertionError):
        call()


@pytest.mark.skipif(torch.cuda.is_available(), reason="an error of a device that is not there")
def test_errors_of_torch_keep_their_types():
    with pytest.raises(torch.AcceleratorError):
        B.lr_linear_fwd(X, WD, WU)


def test_missing_marshalling_fails_loudly(monkeypatch, tmp_path):
    import shutil
    B.lib()
    shutil.copy(B.LIB_PATH, tmp_path / "liblrboost.so")
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "LIB_PATH", str(tmp_path / "liblrboost.so"))
    with pytest.raises(B.LrError):
        B.lr_rms_stat(X)
    # what goes through ctypes does without
    assert B.lr_block_workspace_bytes(DESC, 1) > 0
    with pytest.raises(B.LrError, match="LR_EUNSUPPORTED"):
        B._check(B.lib().lr_rope(16, 128, 16, 16, 1, 4, 1, 128, 0, B.LR_F32, None), "lr_rope")
    monkeypatch.undo()
    with pytest.raises(ValueError):
        B.lr_rms_stat(X[0])


def test_first_calls_of_two_threads(monkeypatch):
    """One thread's first load of the library, ending while the other's marshalling is there already, does not take it away."""
    import sys
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_marshal", None)

    def between_lines(frame, event, arg):
        if frame.f_code is B._native.__code__ and B._marshal is not None:
            B._lib = B._marshal = None      # as the other thread begins
            B.lib()                         # ... and ends
        return between_lines

    before = sys.gettrace()
    sys.settrace(between_lines)
    try:
        m = B._native()
    finally:
        sys.settrace(before)
    assert m is not None
    with pytest.raises(ValueError):
        m.rms_stat(X[0])


def test_library_is_built_without_the_marshalling(monkeypatch):
    """A torch that the marshalling does not compile against fails the build, after the library has been linked."""
    done = []

    def fail():
        raise RuntimeError("no torch headers")

    monkeypatch.setattr(build, "_compile", lambda src: src)
    monkeypatch.setattr(build, "_run", lambda what, cmd: done.append(what))
    monkeypatch.setattr(build, "_compile_marshal", fail)
    with pytest.raises(RuntimeError, match="no torch headers"):
        build.build_library(verbose=False)
    assert done == ["link"]
