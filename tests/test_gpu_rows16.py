"""Forward products of a few rows run as 16 x 16 pieces on a 16 x 16 x 32 matrix instruction: every element has to keep the
bits that the larger tiles, with their 32 x 32 x 16 instruction, give it."""
import pytest
import torch

import launches
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


@pytest.mark.parametrize("t,d_in,r,d_out,pieces", [
    (16, 4096, 1024, 4096, (True, True)),        # 64 and 256 pieces
    (417, 120, 232, 184, (False, False)),        # 405 and 324 of short k
    (141, 208, 512, 456, (False, False)),        # 288 and 261
    (64, 4096, 2048, 1024, (True, True)),        # 512 of long k, 256
    (64, 2048, 2048, 512, (False, True)),        # 512 of 2048 k, 128
    (32, 4096, 4096, 2048, (False, True))])      # 512, but 32 rows of a weight of 4096 rows; 256
def test_second_round_only_for_long_k(t, d_in, r, d_out, pieces):
    """A CU holds one workgroup of 16 x 16 pieces: more than 256 of them take a second round, which long k alone makes up for."""
    x, wd, wu = (torch.zeros(s, dtype=torch.bfloat16, device=DEV) for s in ((t, d_in), (r, d_in), (d_out, r)))
    z, y = (torch.zeros(s, dtype=torch.bfloat16, device=DEV) for s in ((t, r), (t, d_out)))
    assert B.lr_gemm_tile(t, r, d_in, 1, 0, 1) == B.lr_gemm_tile(t, d_out, r, 1, 0, 0) == (32, 32)
    B.lr_linear_fwd_static(x, wd, wu, z, y)      # (its scratch is looked up outside a capture)
    grids = [g for g, _, _ in launches.of(lambda: B.lr_linear_fwd_static(x, wd, wu, z, y))]
    side = [16 if small else 32 for small in pieces]
    assert grids == [-(-t // s) * -(-n // s) for s, n in zip(side, (r, d_out))]
