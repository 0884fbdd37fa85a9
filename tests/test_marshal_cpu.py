"""The native marshalling refuses what the Python one did, with the same kinds of errors, before anything reaches a device."""
import pytest
import torch

from paper_2512_12131_amd import binding as B

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


def test_missing_marshalling_fails_loudly(monkeypatch, tmp_path):
    import shutil
    B.lib()
    shutil.copy(B.LIB_PATH, tmp_path / "liblrboost.so")
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "LIB_PATH", str(tmp_path / "liblrboost.so"))
    with pytest.raises(B.LrError):
        B.lr_rms_stat(X)
