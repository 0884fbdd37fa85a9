"""A backward that is handed no more workspace than it needs, without the room for gathered partials that its query asks for:
the same bits, and nothing written behind the end."""
import ctypes as C

import pytest
import torch

from paper_2512_12131_amd import binding as B
from test_abi_cpu import NEEDED_LINEAR

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 64 << 20      # more than any buffer of the calls: an overrun lands in it


def _run(call, outs, size):
    ws = torch.full((size + GUARD,), 0x5A, dtype=torch.uint8, device=DEV)
    for o in outs:
        o.fill_(0.5)
    status = call(ws.data_ptr(), size)
    torch.cuda.synchronize()
    assert status == 0, f"{size} bytes: status {status}"
    assert bool((ws[size:] == 0x5A).all())
    return [o.clone() for o in outs]


def _same(call, outs, need, query):
    assert need <= query
    for a, b in zip(_run(call, outs, need), _run(call, outs, query)):
        assert torch.equal(a, b)


def _stream():
    return torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("act", [B.LR_ACT_SILU, B.LR_ACT_IDENTITY])
@pytest.mark.parametrize("shape,need", NEEDED_LINEAR)
def test_linear(shape, need, act, accumulate):
    T, d, r, n, dt = shape
    print(f"linear backward in {need} bytes: {shape} act={act} accumulate={accumulate}", flush=True)
    td = torch.bfloat16 if dt == B.LR_BF16 else torch.float32
    g = torch.Generator(device=DEV).manual_seed(T)
    x, wd, wu, dy = (torch.randn(s, generator=g, device=DEV).to(td) for s in ((T, d), (r, d), (n, r), (T, n)))
    z, _ = B.lr_linear_fwd(x, wd, wu, act)
    outs = [torch.empty_like(x), torch.empty((r, d), device=DEV), torch.empty((n, r), device=DEV)]

    def call(ws, size):
        return B.lib().lr_linear_bwd(x.data_ptr(), d, wd.data_ptr(), wu.data_ptr(), z.data_ptr(), dy.data_ptr(), n, outs[0].data_ptr(),
                                     d, outs[1].data_ptr(), outs[2].data_ptr(), T, d, r, n, act, dt, B.LR_F32, accumulate, ws, size,
                                     _stream())

    _same(call, outs, need, B.lr_linear_workspace_bytes(T, d, r, n, dt, 1))


@pytest.mark.parametrize("act", [B.LR_ACT_SILU, B.LR_ACT_IDENTITY])
@pytest.mark.parametrize("norm", [B.LR_NORM_NONE, B.LR_NORM_ONLINE])
@pytest.mark.parametrize("shape,need", [((3, 1031, 264, 40, 520, B.LR_BF16), 782336), ((2, 4, 240, 344, 1480, B.LR_BF16), 2048768),
                                        ((2, 2048, 16, 592, 1240, B.LR_BF16), 16595200), ((3, 300, 72, 24, 104, B.LR_F32), 196352),
                                        ((1, 3844, 264, 488, 2616, B.LR_BF16), 29284352), ((1, 8550, 16, 40, 272, B.LR_BF16), 1509888)])
def test_group(shape, need, norm, act):
    G, T, d, r, n, dt = shape
    print(f"group backward in {need} bytes: {shape} norm={norm} act={act}", flush=True)
    td = torch.bfloat16 if dt == B.LR_BF16 else torch.float32
    g = torch.Generator(device=DEV).manual_seed(T)
    x, wd, wu, dy = (torch.randn(s, generator=g, device=DEV).to(td) for s in ((T, d), (G * r, d), (G, n, r), (G, T, n)))
    gm = torch.ones(d, device=DEV).to(td)
    z, stat, _ = B.lr_group_fwd(x, gm, 1e-5, norm, wd, wu, act)
    outs = [torch.empty_like(x), torch.empty(d, device=DEV), torch.empty((G * r, d), device=DEV), torch.empty((G, n, r), device=DEV)]

    def call(ws, size):
        return B.lib().lr_group_bwd(x.data_ptr(), d, gm.data_ptr(), 1e-5, norm, wd.data_ptr(), wu.data_ptr(), z.data_ptr(),
                                    stat.data_ptr(), dy.data_ptr(), n, T * n, outs[0].data_ptr(), d, outs[1].data_ptr(),
                                    outs[2].data_ptr(), outs[3].data_ptr(), G, T, d, r, n, act, dt, B.LR_F32, 1, ws, size, _stream())

    _same(call, outs, need, B.lr_group_workspace_bytes(G, T, d, r, n, dt, 1))


@pytest.mark.parametrize("form", ["plain", "saved", "lax"])
@pytest.mark.parametrize("shape,need,need_saved", [((2, 256, 2, 2, 344, 64), 6277376, 3905792), ((3, 129, 4, 2, 1003, 136), 9274880, 6135040),
                                                   ((2, 700, 4, 4, 1416, 128), 32633088, 20716032),
                                                   ((8, 770, 1, 1, 2600, 32), 173348608, 77227776)])
def test_block(shape, need, need_saved, form):
    Bn, S, H, kv, f, r = shape
    need = need_saved if form == "saved" else need
    print(f"block backward in {need} bytes: {shape} {form}", flush=True)
    T, d, dkv, f_ld = Bn * S, 128 * H, 128 * kv, (f + 7) // 8 * 8
    g = torch.Generator(device=DEV).manual_seed(S)

    def rand(*s, std=1.0, mean=0.0):
        return (torch.randn(s, generator=g, device=DEV) * std + mean).bfloat16()

    p = {"gamma1": rand(d, std=0.1, mean=1.0), "w_dn_qkv": rand(3 * r, d, std=d ** -0.5), "w_up_qkv": rand(d + 2 * dkv, r, std=r ** -0.5),
         "w_dn_o": rand(r, d, std=d ** -0.5), "w_up_o": rand(d, r, std=r ** -0.5), "gamma2": rand(d, std=0.1, mean=1.0),
         "w_dn_gu": rand(2 * r, d, std=d ** -0.5), "w_up_gu": rand(2, f_ld, r, std=r ** -0.5), "w_dn_d": rand(r, f_ld, std=f ** -0.5),
         "w_up_d": rand(d, r, std=r ** -0.5)}
    p["w_up_gu"][:, f:] = 0
    p["w_dn_d"][:, f:] = 0
    desc = B.make_block_desc(Bn, S, d, H, 128, f, f_ld, r, act=B.LR_ACT_IDENTITY if form == "lax" else B.LR_ACT_SILU, n_kv_heads=kv)
    x, dy = rand(T, d), rand(T, d)
    dx = torch.empty_like(x)
    grads = {n: torch.empty_like(t, dtype=torch.float32) for n, t in p.items()}
    ps, gs = B._params_struct(p), B._params_struct(grads)
    saved = B.alloc_block_saved(desc, x.device)
    if form == "saved":
        _, ck, saved = B.lr_block_fwd_save(desc, p, x, saved=saved)
    elif form == "lax":
        _, ck = B.lr_block_lax_fwd(desc, p, x)
    else:
        _, ck = B.lr_block_fwd(desc, p, x)
    cs, ss, lx = B._ckpt_struct(ck), B._saved_struct(saved), B._lax_struct()
    lib = B.lib()

    def call(ws, size):
        a = (C.byref(desc), C.byref(ps), x.data_ptr(), dy.data_ptr(), C.byref(cs))
        if form == "saved":
            return lib.lr_block_bwd_saved(*a, C.byref(ss), dx.data_ptr(), C.byref(gs), 1, ws, size, _stream())
        if form == "lax":
            return lib.lr_block_lax_bwd(*a, dx.data_ptr(), C.byref(gs), 1, C.byref(lx), ws, size, _stream())
        return lib.lr_block_bwd(*a, dx.data_ptr(), C.byref(gs), 1, ws, size, _stream())

    query = lib.lr_block_saved_workspace_bytes(C.byref(desc), 1) if form == "saved" else B.lr_block_workspace_bytes(desc, 1)
    _same(call, [dx, *grads.values()], need, query)


@pytest.mark.parametrize("f", [2600, 2624, 1376])     # rows that get room up to a cache line, that end on one, that would grow by 2 %
def test_block_without_room_for_rows_on_cache_lines(f):
    """Forward and backward in the query's size less the ends of g, u, m, dg and du: accepted, the same bits, nothing past the end."""
    Bn, S, H, r = 2, 640, 4, 136
    T, d, pad = Bn * S, 128 * H, 24 if f == 2600 else 0
    print(f"block in the room of unpadded rows, f={f}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(f)
    shapes = {"gamma1": (d,), "w_dn_qkv": (3 * r, d), "w_up_qkv": (3, d, r), "w_dn_o": (r, d), "w_up_o": (d, r), "gamma2": (d,),
              "w_dn_gu": (2 * r, d), "w_up_gu": (2, f, r), "w_dn_d": (r, f), "w_up_d": (d, r)}
    p = {n: (torch.randn(s, generator=g, device=DEV) * s[-1] ** -0.5).bfloat16() for n, s in shapes.items()}
    x, dy = (torch.randn((T, d), generator=g, device=DEV).bfloat16() for _ in range(2))
    desc = B.make_block_desc(Bn, S, d, H, 128, f, f, r)
    lib, ps, ck, y, dx = B.lib(), B._params_struct(p), B.alloc_block_ckpt(desc, x.device), torch.empty_like(x), torch.empty_like(x)
    grads = {n: torch.empty_like(t, dtype=torch.float32) for n, t in p.items()}
    cs, gs = B._ckpt_struct(ck), B._params_struct(grads)

    def fwd(ws, size):
        return lib.lr_block_fwd(C.byref(desc), C.byref(ps), x.data_ptr(), y.data_ptr(), C.byref(cs), ws, size, _stream())

    def bwd(ws, size):
        return lib.lr_block_bwd(C.byref(desc), C.byref(ps), x.data_ptr(), dy.data_ptr(), C.byref(cs), dx.data_ptr(), C.byref(gs), 1, ws, size,
                                _stream())

    for call, outs, rows in ((fwd, [y, *ck.values()], 2), (bwd, [dx, *grads.values()], 5)):
        query = B.lr_block_workspace_bytes(desc, int(call is bwd))
        _same(call, outs, query - rows * T * pad * 2, query)


def test_saved_backward_uses_the_room_for_rows_on_cache_lines():
    """What the query asks for the ends of dg's and du's rows is taken up by them: no more whole 64 bytes stay untouched than without."""
    Bn, S, H, f, r = 8, 770, 1, 2600, 344
    T, d, pad = Bn * S, 128 * H, 24
    print(f"kept-activation backward, what it leaves untouched, f={f}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(f)
    shapes = {"gamma1": (d,), "w_dn_qkv": (3 * r, d), "w_up_qkv": (3, d, r), "w_dn_o": (r, d), "w_up_o": (d, r), "gamma2": (d,),
              "w_dn_gu": (2 * r, d), "w_up_gu": (2, f, r), "w_dn_d": (r, f), "w_up_d": (d, r)}
    p = {n: (torch.randn(s, generator=g, device=DEV) * s[-1] ** -0.5).bfloat16() for n, s in shapes.items()}
    x, dy = (torch.randn((T, d), generator=g, device=DEV).bfloat16() for _ in range(2))
    desc = B.make_block_desc(Bn, S, d, H, 128, f, f, r)
    _, ck, saved = B.lr_block_fwd_save(desc, p, x)
    query = B.lib().lr_block_saved_workspace_bytes(C.byref(desc), 1)
    outs, untouched = [], []
    for size in (query, query - 2 * T * pad * 2):
        ws = torch.full((size,), 0x55, dtype=torch.uint8, device=DEV)
        dx, grads = torch.empty_like(x), {n: torch.empty_like(t, dtype=torch.float32) for n, t in p.items()}
        status = B.lib().lr_block_bwd_saved(C.byref(desc), C.byref(B._params_struct(p)), x.data_ptr(), dy.data_ptr(),
                                            C.byref(B._ckpt_struct(ck)), C.byref(B._saved_struct(saved)), dx.data_ptr(),
                                            C.byref(B._params_struct(grads)), 0, ws.data_ptr(), size, _stream())
        torch.cuda.synchronize()
        assert status == 0
        outs.append([dx, *grads.values()])
        untouched.append(64 * int((ws[:size // 64 * 64].view(-1, 64) == 0x55).all(1).sum()))
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    assert untouched[0] - untouched[1] < T * pad * 2, untouched


def test_rows_that_span_more_than_2_gib():
    """x and dy as columns of a 2.6 GB tensor: refused in the workspace of dense rows, and with the room for copies the gradients of
    dense rows.  Each is a chained sum of T exact products in both: off by at most T 2^-24 of the sum of their magnitudes."""
    T, d, r, n, wide = 65536, 64, 16, 72, 20000
    print("layer backward over rows that span 2.6 GB", flush=True)
    g = torch.Generator(device=DEV).manual_seed(1)
    big = torch.empty((T, wide), dtype=torch.bfloat16, device=DEV)
    x, dy = big[:, 8:8 + d], big[:, 512:512 + n]
    x.copy_(torch.randn((T, d), generator=g, device=DEV))
    dy.copy_(torch.randn((T, n), generator=g, device=DEV))
    wd, wu = torch.randn((r, d), generator=g, device=DEV).bfloat16(), torch.randn((n, r), generator=g, device=DEV).bfloat16()
    z, _ = B.lr_linear_fwd(x, wd, wu, B.LR_ACT_IDENTITY)
    outs = [torch.empty((T, d), dtype=torch.bfloat16, device=DEV), torch.empty((r, d), device=DEV), torch.empty((n, r), device=DEV)]

    def call(ws, size):
        return B.lib().lr_linear_bwd(x.data_ptr(), wide, wd.data_ptr(), wu.data_ptr(), z.data_ptr(), dy.data_ptr(), wide,
                                     outs[0].data_ptr(), d, outs[1].data_ptr(), outs[2].data_ptr(), T, d, r, n, B.LR_ACT_IDENTITY,
                                     B.LR_BF16, B.LR_F32, 0, ws, size, _stream())

    query = B.lr_linear_workspace_bytes(T, d, r, n, B.LR_BF16, 1)
    ws = torch.empty(query, dtype=torch.uint8, device=DEV)
    assert call(ws.data_ptr(), query) == -3
    got = _run(call, outs, query + T * (n + r) * 2 + 4096)
    dense = B.lr_linear_bwd(x.contiguous(), wd, wu, z, dy.contiguous(), B.LR_ACT_IDENTITY)
    assert torch.equal(got[0], dense[0])
    dz = (dy.double() @ wu.double()).bfloat16().double()
    for a, b, mag in ((got[1], dense[1], dz.abs().t() @ x.double().abs()), (got[2], dense[2], dy.double().abs().t() @ z.double().abs())):
        assert ((a.double() - b.double()).abs() <= 2 * T * 2.0 ** -24 * 1.01 * mag).all()


# the score gradient formed twice (no room for it in the workspace) and stored, key / value heads of groups behind it
@pytest.mark.parametrize("Bn,S,H,Hkv", [(8, 264, 20, 20), (9, 264, 20, 10), (3, 264, 20, 10), (1, 520, 4, 2), (2, 333, 4, 4)])
def test_attention(Bn, S, H, Hkv):
    print(f"attention backward in the bytes of its query B={Bn} S={S} H={H} Hkv={Hkv}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(S)
    q, dout = (torch.randn((Bn * S, H * 128), generator=g, device=DEV).bfloat16() for _ in range(2))
    k, v = (torch.randn((Bn * S, Hkv * 128), generator=g, device=DEV).bfloat16() for _ in range(2))
    o, lse = B.lr_attention_gqa_fwd(q, k, v, Bn, S, H, Hkv, 128)
    outs = [torch.empty_like(t) for t in (q, k, v)]

    def call(ws, size):
        return B.lib().lr_attention_gqa_bwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), dout.data_ptr(), lse.data_ptr(),
                                            *(t.data_ptr() for t in outs), H * 128, Hkv * 128, Bn, S, H, Hkv, 128, 1, B.LR_BF16, ws, size,
                                            _stream())

    need = B.lib().lr_attention_gqa_bwd_workspace_bytes(Bn, S, H, Hkv, 128)
    _same(call, outs, need, need + Bn * H * S * S * 2)
    for a, b in zip(outs, B.lr_attention_gqa_bwd(q, k, v, o, dout, lse, Bn, S, H, Hkv, 128)):
        assert torch.equal(a, b)
