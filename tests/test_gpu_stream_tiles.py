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


# the LaX forms (z + h handed on; the gradient's sum with the one from above): several tiles per workgroup, remainders of rows and columns; long k
@pytest.mark.parametrize("n,S,H,f,r", [(136, 120, 1, 344, 520), (72, 127, 8, 2760, 200)])
def test_lax_rows(n, S, H, f, r):
    print(f"stream of 128 x 128 tiles, LaX B={n} S={S} H={H} f={f} r={r}", flush=True)
    T, d, few = n * S, 128 * H, 2
    g = torch.Generator(device=DEV).manual_seed(r)
    rand = lambda *shape, std=1.0, mean=0.0: (torch.randn(shape, generator=g, device=DEV) * std + mean).bfloat16()
    p = {"gamma1": rand(d, std=0.1, mean=1.0), "w_dn_qkv": rand(3 * r, d, std=d ** -0.5), "w_up_qkv": rand(3, d, r, std=r ** -0.5),
         "w_dn_o": rand(r, d, std=d ** -0.5), "w_up_o": rand(d, r, std=r ** -0.5), "gamma2": rand(d, std=0.1, mean=1.0),
         "w_dn_gu": rand(2 * r, d, std=d ** -0.5), "w_up_gu": rand(2, f, r, std=r ** -0.5), "w_dn_d": rand(r, f, std=f ** -0.5),
         "w_up_d": rand(d, r, std=r ** -0.5)}
    x, dy = rand(T, d), rand(T, d)
    h, dz = ({k: rand(T, m * r) for k, m in (("qkv", 3), ("o", 1), ("gu", 2), ("d", 1))} for _ in range(2))
    desc = lambda b: B.make_block_desc(b, S, d, H, 128, f, f, r, act=B.LR_ACT_IDENTITY)
    head = lambda t: {k: v[:few * S] for k, v in t.items()} if isinstance(t, dict) else t[:few * S]

    forward = lambda: B.lr_block_lax_fwd(desc(n), p, x, h)
    y, ck = forward()
    backward = lambda: B.lr_block_lax_bwd(desc(n), p, x, dy, ck, h, dz)
    dx, _, dh = backward()
    y1, ck1 = B.lr_block_lax_fwd(desc(few), p, head(x), head(h))
    dx1, _, dh1 = B.lr_block_lax_bwd(desc(few), p, head(x), head(dy), ck1, head(h), head(dz))
    torch.cuda.synchronize()
    assert torch.equal(y1, head(y)) and torch.equal(dx1, head(dx))
    for a, b in ((ck1, ck), (dh1, dh)):
        for k in a:
            assert torch.equal(a[k], b[k][:few * S])
    # (8: z + h, 9: its gradient)
    assert len([*launches.named(forward, "gemm_stream_kernelILi8ELb0E")]) and len([*launches.named(backward, "gemm_stream_kernelILi9ELb1E")])
