"""Errors of the native marshalling that show only where there is a device."""
import pytest
import torch

from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_no_room_for_an_output_is_torchs_own_error():
    x, wd, row = (torch.zeros(s, device=DEV) for s in ((16, 8), (8, 8), (1, 8)))
    with pytest.raises(torch.OutOfMemoryError):
        B.lr_linear_fwd(x, wd, row.expand(1 << 40, 8))
