"""128 x 128 tiles as a stream: a workgroup walks several tiles, the stages of the next one under way during an epilogue; or one tile
each where k is long.  Rows have the bits of calls on few tokens, which run on other tiles."""
import pytest
import torch

import launches
from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LDS = 2 * (128 + 128) * 128 + 4 * 4096      # of a workgroup: two stages, and staging space for the epilogue


# which of z, y (forward) and dx (backward) run as a stream; k of one slice, of two with a remainder, of an odd number, remainders of rows
# and columns, members, more than two tiles per workgroup and one at most
@pytest.mark.parametrize("T,d,r,n,G,streams", [(16300, 264, 64, 520, 1, "y"), (9000, 520, 72, 1032, 2, "y"), (5000, 2000, 384, 2048, 2, "y"),
                                               (8200, 1096, 264, 1096, 3, "z"), (2500, 2048, 1024, 512, 2, "z dx")])
def test_rows(T, d, r, n, G, streams):
    print(f"stream of 128 x 128 tiles T={T} d={d} r={r} n={n} G={G}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(T)
    x, dy = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((T, d), (G, T, n)))
    wd = (torch.randn((G * r, d), generator=g, device=DEV) * d ** -0.5).bfloat16()
    wu = (torch.randn((G, n, r), generator=g, device=DEV) * r ** -0.5).bfloat16()
    gamma = torch.ones(d, device=DEV).bfloat16()

    def forward(rows):
        z, _, y = B.lr_group_fwd(x[rows], gamma, 1e-5, B.LR_NORM_NONE, wd, wu)
        return z, y

    def backward(rows, z):
        return B.lr_group_bwd(x[rows], gamma, 1e-5, B.LR_NORM_NONE, wd, wu, z, torch.ones(z.shape[0], device=DEV), dy[:, rows].contiguous())[0]

    whole = slice(0, T)
    z, y = forward(whole)
    dx = backward(whole, z)
    for rows in (slice(0, 200), slice(T - 200, T)):
        z1, y1 = forward(rows)
        dx1 = backward(rows, z1)
        torch.cuda.synchronize()
        assert torch.equal(z1, z[rows]) and torch.equal(y1, y[:, rows]) and torch.equal(dx1, dx[rows])
    is_stream = [k[1:] == (256, LDS) for k in launches.of(lambda: forward(whole))]
    assert is_stream == ["z" in streams, "y" in streams]
    assert ("dx" in streams) == ((256, LDS) in [k[1:] for k in launches.of(lambda: backward(whole, z))][-1:])
