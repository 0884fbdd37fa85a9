"""The three products at the end of a layer's backward run in one launch where they are small.  While launches are being timed each
has its own, and added to zeros instead of written the weight gradients go through a finishing pass: every output has to have the
same bits."""
import pytest
import torch

import launches
from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _both(T, d_in, r, d_out, dt, act, grad_dt):
    g = torch.Generator().manual_seed(T + r)
    x, wd, wu, dy = (torch.randn(s, generator=g).to(dt).to(DEV) for s in ((T, d_in), (r, d_in), (d_out, r), (T, d_out)))
    z, y = B.lr_linear_fwd(x, wd, wu, act)
    plain = B.lr_linear_bwd(x, wd, wu, z, dy, act, grad_dt=grad_dt)
    gt = torch.float32 if grad_dt == B.LR_F32 else torch.bfloat16
    zeros = tuple(torch.zeros(w.shape, dtype=gt, device=DEV) for w in (wd, wu))
    added = B.lr_linear_bwd(x, wd, wu, z, dy, act, grads=zeros, grad_dt=grad_dt)
    torch.cuda.synchronize()
    B.lr_launch_timer_begin(16)
    apart = B.lr_linear_bwd(x, wd, wu, z, dy, act, grad_dt=grad_dt)
    torch.cuda.synchronize()
    records = B.lr_launch_timer_end()
    assert dt == torch.float32 or len(records) == 4      # (the timer sees, and keeps apart, bf16 products)
    return (x, wd, wu, dy, z), plain, added, apart


@pytest.mark.parametrize("grad_dt", [B.LR_F32, B.LR_BF16])
@pytest.mark.parametrize("act", [B.LR_ACT_SILU, B.LR_ACT_IDENTITY])
@pytest.mark.parametrize("T,d_in,r,d_out", [(1, 8, 8, 8), (31, 40, 24, 72), (32, 64, 32, 64), (33, 128, 40, 96), (65, 256, 64, 24),
                                            (513, 264, 72, 520), (1031, 1024, 256, 768), (2050, 512, 128, 512)])
def test_bf16(T, d_in, r, d_out, act, grad_dt):
    print(f"joint bf16 T={T} {d_in}->{r}->{d_out} act={act}", flush=True)
    _, plain, added, apart = _both(T, d_in, r, d_out, torch.bfloat16, act, grad_dt)
    for a, b, c in zip(plain, added, apart):
        assert torch.equal(a, b) and torch.equal(a, c)


@pytest.mark.parametrize("act", [B.LR_ACT_SILU, B.LR_ACT_IDENTITY])
@pytest.mark.parametrize("T,d_in,r,d_out", [(1, 1, 1, 1), (31, 33, 5, 7), (64, 32, 32, 96), (129, 127, 33, 65), (512, 256, 64, 256),
                                            (1023, 511, 127, 509)])
def test_f32(T, d_in, r, d_out, act):
    """... and in 32 bits against 64: each gradient is one or two chained sums, and n terms added in 32 bits are off by at most
    n 2^-24 times the sum of their magnitudes; the tested lengths stay below 2^11, in practice far below the bound."""
    print(f"joint f32 T={T} {d_in}->{r}->{d_out} act={act}", flush=True)
    (x, wd, wu, dy, z), plain, added, _ = _both(T, d_in, r, d_out, torch.float32, act, B.LR_F32)
    for a, b in zip(plain, added):
        assert torch.equal(a, b)
    x, wd, wu, dy, z = (t.double().cpu() for t in (x, wd, wu, dy, z))
    s = torch.sigmoid(z)
    sig, prime = (z * s, s * (1 + z * (1 - s))) if act == B.LR_ACT_SILU else (z, torch.ones_like(z))
    dz = (dy @ wu) * prime
    for got, ref in zip(plain, (dz @ wd, dz.t() @ x, dy.t() @ sig)):
        assert (got.double().cpu() - ref).norm() <= 2.0 ** 11 * 2.0 ** -24 * ref.norm()


@pytest.mark.parametrize("Bn,S,H,kv,f,r,lax,grad_dt", [(2, 256, 2, 2, 344, 64, False, B.LR_F32), (1, 33, 1, 1, 200, 40, False, B.LR_BF16),
                                                       (3, 129, 4, 2, 1003, 136, False, B.LR_F32), (1, 520, 4, 1, 1416, 128, True, B.LR_F32),
                                                       (2, 500, 8, 8, 2730, 256, False, B.LR_BF16)])
def test_block(Bn, S, H, kv, f, r, lax, grad_dt):
    """A block's backward with its independent products joined, and (while launches are being timed) each on its own."""
    print(f"joint block B={Bn} S={S} H={H}/{kv} f={f} r={r} lax={lax}", flush=True)
    T, d, dkv, f_ld = Bn * S, 128 * H, 128 * kv, (f + 7) // 8 * 8
    g = torch.Generator(device=DEV).manual_seed(S)

    def rand(*shape, std=1.0, mean=0.0):
        return (torch.randn(shape, generator=g, device=DEV) * std + mean).bfloat16()

    p = {"gamma1": rand(d, std=0.1, mean=1.0), "w_dn_qkv": rand(3 * r, d, std=d ** -0.5), "w_up_qkv": rand(d + 2 * dkv, r, std=r ** -0.5),
         "w_dn_o": rand(r, d, std=d ** -0.5), "w_up_o": rand(d, r, std=r ** -0.5), "gamma2": rand(d, std=0.1, mean=1.0),
         "w_dn_gu": rand(2 * r, d, std=d ** -0.5), "w_up_gu": rand(2, f_ld, r, std=r ** -0.5), "w_dn_d": rand(r, f_ld, std=f ** -0.5),
         "w_up_d": rand(d, r, std=r ** -0.5)}
    p["w_up_gu"][:, f:] = 0
    p["w_dn_d"][:, f:] = 0
    desc = B.make_block_desc(Bn, S, d, H, 128, f, f_ld, r, act=B.LR_ACT_IDENTITY if lax else B.LR_ACT_SILU, grad_dt=grad_dt, n_kv_heads=kv)
    x, dy = rand(T, d), rand(T, d)
    if lax:
        wide = {"qkv": 3, "o": 1, "gu": 2, "d": 1}
        hp, dz = ({n: rand(T, w * r) for n, w in wide.items()} for _ in range(2))
        _, ck = B.lr_block_lax_fwd(desc, p, x, h_prev=hp)

    def backward():
        if lax:
            dx, grads, dh = B.lr_block_lax_bwd(desc, p, x, dy, ck, h_prev=hp, dz_next=dz)
            return {"dx": dx, **grads, **{"dh_" + n: t for n, t in dh.items()}}
        dx, grads = B.lr_block_bwd(desc, p, x, dy, ck)
        return {"dx": dx, **grads}

    if not lax:
        _, ck = B.lr_block_fwd(desc, p, x)
    joined = backward()
    B.lr_launch_timer_begin(200)
    apart = backward()
    torch.cuda.synchronize()
    B.lr_launch_timer_end()
    off = [n for n, t in joined.items() if not torch.equal(t, apart[n])]
    assert not off, off


@pytest.mark.parametrize("grad_dt", [B.LR_F32, B.LR_BF16])
@pytest.mark.parametrize("G,T,d_in,r,d_out", [(1, 1024, 64, 32, 72), (1, 1031, 264, 40, 520), (1, 2113, 8, 8, 8), (3, 1700, 256, 64, 256),
                                              (2, 5120, 256, 64, 616), (14, 1100, 64, 16, 72), (2, 8192, 1024, 512, 1024)])
def test_gathered_gradients(G, T, d_in, r, d_out, grad_dt):
    """Split weight gradients summed up in one launch at the end: sizes at and above two splits, that end within a workgroup,
    more gradients than one launch takes, and partials that do not all fit the region they are gathered in.  sigma = identity,
    so dW_up is a chained sum of exact products: off by at most T 2^-24 of the sum of their magnitudes, and a bf16 rounding."""
    print(f"gathered G={G} T={T} {d_in}->{r}->{d_out}", flush=True)
    g = torch.Generator().manual_seed(T)
    x, wd, wu, dy = (torch.randn(s, generator=g).bfloat16().to(DEV) for s in ((T, d_in), (G * r, d_in), (G, d_out, r), (G, T, d_out)))
    gt = torch.float32 if grad_dt == B.LR_F32 else torch.bfloat16
    base = [torch.randn(s, generator=g).to(gt).to(DEV) for s in ((G * r, d_in), (G, d_out, r))]
    if G == 1:
        z, _ = B.lr_linear_fwd(x, wd, wu[0], B.LR_ACT_IDENTITY)
        run = lambda grads: B.lr_linear_bwd(x, wd, wu[0], z, dy[0], B.LR_ACT_IDENTITY, grads=grads, grad_dt=grad_dt)
        _, dwd, dwu = run(None)
        _, awd, awu = run((base[0].clone(), base[1][0].clone()))
        dwu, awu = dwu[None], awu[None]
    else:
        gm = torch.ones(d_in, device=DEV).bfloat16()
        z, stat, _ = B.lr_group_fwd(x, gm, 1e-5, B.LR_NORM_NONE, wd, wu, B.LR_ACT_IDENTITY)
        run = lambda grads: B.lr_group_bwd(x, gm, 1e-5, B.LR_NORM_NONE, wd, wu, z, stat, dy, B.LR_ACT_IDENTITY, grads=grads,
                                           grad_dt=grad_dt)
        _, _, dwd, dwu = run(None)
        _, _, awd, awu = run((torch.zeros(d_in, dtype=gt, device=DEV), base[0].clone(), base[1].clone()))
    for i in range(G):
        a, b = dy[i].double().cpu(), z[:, i * r:(i + 1) * r].double().cpu()
        bound = (a.abs().t() @ b.abs()) * (T * 2.0 ** -24)
        ref = a.t() @ b
        if grad_dt == B.LR_BF16:
            bound = bound + (ref.abs() + bound) * 2.0 ** -8
        assert ((dwu[i].double().cpu() - ref).abs() <= bound).all()
    if grad_dt == B.LR_F32:   # added to what is there: the same sum and one more rounding
        assert torch.equal(awd, dwd + base[0]) and torch.equal(awu, dwu + base[1])


@pytest.mark.parametrize("grad_dt", [B.LR_F32, B.LR_BF16])
@pytest.mark.parametrize("G,T,d_in,r,d_out", [(1, 1024, 64, 32, 72), (1, 1031, 264, 40, 520), (1, 2113, 8, 8, 8), (3, 1700, 256, 64, 256),
                                              (2, 5120, 256, 64, 616), (14, 1100, 64, 16, 72), (2, 8192, 1024, 512, 1024)])
def test_gathered_gradients_against_64_bits(G, T, d_in, r, d_out, grad_dt):
    """All gradients, written and added.  W_up picks a column of dy for each of dz, which is then exact, so both gradients are chained
    sums of exact products: off by at most T 2^-24 of the sum of their magnitudes, one more 32-bit rounding where they are added to
    what is there, and a bf16 rounding."""
    print(f"gathered, 64 bits G={G} T={T} {d_in}->{r}->{d_out}", flush=True)
    g = torch.Generator().manual_seed(T + 1)
    x, wd, dy = (torch.randn(s, generator=g).bfloat16().to(DEV) for s in ((T, d_in), (G * r, d_in), (G, T, d_out)))
    pick = torch.stack([torch.randperm(d_out, generator=g)[:r] for _ in range(G)])
    wu = torch.zeros((G, d_out, r), dtype=torch.bfloat16)
    wu[torch.arange(G)[:, None], pick, torch.arange(r)[None, :]] = 1
    wu = wu.to(DEV)
    gt = torch.float32 if grad_dt == B.LR_F32 else torch.bfloat16
    base = [torch.randn(s, generator=g).to(gt).to(DEV) for s in ((G * r, d_in), (G, d_out, r))]
    if G == 1:
        z, _ = B.lr_linear_fwd(x, wd, wu[0], B.LR_ACT_IDENTITY)
        run = lambda grads: B.lr_linear_bwd(x, wd, wu[0], z, dy[0], B.LR_ACT_IDENTITY, grads=grads, grad_dt=grad_dt)[1:]
        got = [run(None), run((base[0].clone(), base[1][0].clone()))]
        got = [(down, up[None]) for down, up in got]
    else:
        gm = torch.ones(d_in, device=DEV).bfloat16()
        z, stat, _ = B.lr_group_fwd(x, gm, 1e-5, B.LR_NORM_NONE, wd, wu, B.LR_ACT_IDENTITY)
        run = lambda grads: B.lr_group_bwd(x, gm, 1e-5, B.LR_NORM_NONE, wd, wu, z, stat, dy, B.LR_ACT_IDENTITY, grads=grads,
                                           grad_dt=grad_dt)[2:]
        got = [run(None), run((torch.zeros(d_in, dtype=gt, device=DEV), base[0].clone(), base[1].clone()))]
    for i in range(G):
        dz = dy[i][:, pick[i].to(DEV)]
        rows = slice(i * r, (i + 1) * r)
        for a, b, outs in ((dz, x, [(down[rows], add) for (down, _), add in zip(got, (None, base[0][rows]))]),
                           (dy[i], z[:, rows], [(up[i], add) for (_, up), add in zip(got, (None, base[1][i]))])):
            a, b = a.double(), b.double()
            ref, mag = a.t() @ b, a.abs().t() @ b.abs()
            for out, add in outs:
                want, bound = ref, mag * (T * 2.0 ** -24)
                if add is not None:
                    want = ref + add.double()
                    bound = bound + (want.abs() + bound) * 2.0 ** -24
                if grad_dt == B.LR_BF16:
                    bound = bound + (want.abs() + bound) * 2.0 ** -8
                assert ((out.double() - want).abs() <= bound).all()


BF, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("T,d_in,r,d_out,dt,count", [
    (16, 1024, 256, 1024, BF, 2), (33, 128, 40, 96, BF, 2), (513, 264, 72, 520, BF, 2), (1031, 1024, 256, 768, BF, 2),   # dz, then the rest
    (2050, 512, 128, 512, BF, 3),                                                             # ... and a finishing pass
    (3380, 2088, 72, 72, BF, 5),                                                              # apart: faster so
    (33, 128, 40, 96, F32, 2), (512, 256, 64, 256, F32, 2), (513, 264, 72, 520, F32, 2),
    (16, 1024, 256, 1024, F32, 4), (1031, 1024, 256, 768, F32, 4)])                           # more than 512 tiles
def test_launches_of_a_layer_backward(T, d_in, r, d_out, dt, count):
    x, wd, wu, dy, z = (torch.zeros(s, dtype=dt, device=DEV) for s in ((T, d_in), (r, d_in), (d_out, r), (T, d_out), (T, r)))
    assert len(launches.of(lambda: B.lr_linear_bwd(x, wd, wu, z, dy))) == count
