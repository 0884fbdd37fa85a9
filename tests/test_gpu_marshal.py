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


def test_half_of_the_gradients_is_refused():
    """... by the library, before any launch: given gradients are added to, and there is nothing to add to."""
    T, d, r, n = 16, 32, 8, 24
    x, wd, wu, z, dy = (torch.zeros(s, device=DEV) for s in ((T, d), (r, d), (n, r), (T, r), (T, n)))
    gd, gu, gamma, stat = (torch.zeros(s, device=DEV) for s in ((r, d), (n, r), (d,), (T,)))
    for grads in ((None, gu), (gd, None), (None, None)):
        with pytest.raises(B.LrError):
            B.lr_linear_bwd(x, wd, wu, z, dy, grads=grads)
    for grads in ((None, gd, gu[None]), (gamma, None, gu[None]), (gamma, gd, None)):
        with pytest.raises(B.LrError):
            B.lr_group_bwd(x, gamma, 1e-5, B.LR_NORM_ONLINE, wd, wu[None], z, stat, dy[None], grads=grads)
