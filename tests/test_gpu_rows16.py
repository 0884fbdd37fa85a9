"""Forward products of a few rows run as 16 x 16 pieces on a 16 x 16 x 32 matrix instruction: every element has to keep the
bits that the larger tiles, with their 32 x 32 x 16 instruction, give it."""
import pytest
import torch

from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T_FULL = 4096


def _bf(g, *shape):
    # a spread of magnitudes: sums that cancel, terms that vanish beside others
    t = torch.randn(shape, generator=g, device=DEV) * torch.exp2(torch.randint(-12, 13, shape, generator=g, device=DEV).float())
    return t.bfloat16()


@pytest.mark.parametrize("act", [B.LR_ACT_SILU, B.LR_ACT_IDENTITY])
@pytest.mark.parametrize("d_in,r,d_out", [(8, 8, 8), (64, 16, 24), (72, 24, 1000), (256, 64, 40), (520, 136, 264), (1032, 72, 520),
                                          (4096, 264, 1032)])
def test_rows_of_a_layer(d_in, r, d_out, act):
    g = torch.Generator(device=DEV).manual_seed(d_in + r)
    x, wd, wu = _bf(g, T_FULL, d_in), _bf(g, r, d_in), _bf(g, d_out, r)
    z, y = B.lr_linear_fwd(x, wd, wu, act)
    for t in (1, 7, 15, 16, 17, 31, 33, 48, 64, 97):
        print(f"rows16 {d_in}->{r}->{d_out} t={t}", flush=True)
        z1, y1 = B.lr_linear_fwd(x[:t].contiguous(), wd, wu, act)
        assert torch.equal(z1.view(torch.int16), z[:t].view(torch.int16))
        assert torch.equal(y1.view(torch.int16), y[:t].view(torch.int16))


@pytest.mark.parametrize("norm", [B.LR_NORM_NONE, B.LR_NORM_ONLINE, B.LR_NORM_TWO_PASS])
def test_rows_of_a_group(norm):
    d, r, n, G = 776, 264, 136, 3
    g = torch.Generator(device=DEV).manual_seed(9)
    x, wd, wu = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((T_FULL, d), (G * r, d), (G, n, r)))
    gamma = (1 + 0.1 * torch.randn((d,), generator=g, device=DEV)).bfloat16()
    z, _, y = B.lr_group_fwd(x, gamma, 1e-5, norm, wd, wu)
    for t in (1, 16, 33, 64):
        z1, _, y1 = B.lr_group_fwd(x[:t].contiguous(), gamma, 1e-5, norm, wd, wu)
        assert torch.equal(z1, z[:t]) and torch.equal(y1, y[:, :t])
