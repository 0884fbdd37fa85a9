"""Operands that are column slices of a wider tensor (q, k and v of one product, gate and up of one product): every output has the bits
of the call on dense copies, in memory of its own whose rows are as far apart as the input's."""
import pytest
import torch

from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _slices(rows, widths, seed):
    """Slices of one wide tensor, with columns of nobody before and after each."""
    gap = 24
    g = torch.Generator(device=DEV).manual_seed(seed)
    wide = torch.randn((rows, sum(widths) + gap * (len(widths) + 1)), generator=g, device=DEV).bfloat16()
    at, out = gap, []
    for w in widths:
        out.append(wide[:, at:at + w])
        at += w + gap
    return out


def _check(got, want):
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


# one token, ragged lengths (score gradient formed twice), lengths of whole vectors (stored), and many heads of them (formed twice)
@pytest.mark.parametrize("Bn,S,H,Hkv", [(1, 1, 1, 1), (2, 200, 2, 1), (1, 333, 4, 4), (2, 264, 4, 2), (8, 264, 20, 20)])
def test_attention(Bn, S, H, Hkv):
    print(f"padded rows, attention B={Bn} S={S} H={H} Hkv={Hkv}", flush=True)
    q, k, v, dout = _slices(Bn * S, [H * 128, Hkv * 128, Hkv * 128, H * 128], S)
    qd, kd, vd, dd = (t.contiguous() for t in (q, k, v, dout))
    o, lse = B.lr_attention_gqa_fwd(q, k, v, Bn, S, H, Hkv, 128)
    od, lsed = B.lr_attention_gqa_fwd(qd, kd, vd, Bn, S, H, Hkv, 128)
    _check([o, lse], [od, lsed])
    want = B.lr_attention_gqa_bwd(qd, kd, vd, od, dd, lsed, Bn, S, H, Hkv, 128)
    _check(B.lr_attention_gqa_bwd(q, k, v, o, dout, lse, Bn, S, H, Hkv, 128), want)
    if H == Hkv:
        o, lse = B.lr_attention_fwd(q, k, v, Bn, S, H, 128)
        _check([o, lse], [od, lsed])
        _check(B.lr_attention_bwd(q, k, v, o, dout, lse, Bn, S, H, 128), want)


@pytest.mark.parametrize("T,f", [(1, 8), (33, 200), (1031, 1376)])
def test_swiglu(T, f):
    print(f"padded rows, swiglu T={T} f={f}", flush=True)
    g, u, dm = _slices(T, [f, f, f], f)
    dense = [t.contiguous() for t in (g, u, dm)]
    _check([B.lr_swiglu_fwd(g, u)], [B.lr_swiglu_fwd(*dense[:2])])
    _check(B.lr_swiglu_bwd(g, u, dm), B.lr_swiglu_bwd(*dense))


def test_dense_operands_of_other_shapes():
    """[B, S, H, 128], or the rows of all heads one after the other, is the memory of dense [B * S, H * 128]."""
    Bn, S, H = 2, 40, 3
    print(f"operands by sequences and heads B={Bn} S={S} H={H}", flush=True)
    q, k, v, dout = (t.contiguous() for t in _slices(Bn * S, [H * 128] * 4, S))
    heads, rows = (lambda t: t.view(Bn, S, H, 128)), (lambda t: t.view(Bn * S * H, 128))
    o, lse = B.lr_attention_fwd(q, k, v, Bn, S, H, 128)
    _check(B.lr_attention_fwd(q, heads(k), rows(v), Bn, S, H, 128), [o, lse])
    want = B.lr_attention_gqa_bwd(q, k, v, o, dout, lse, Bn, S, H, H, 128)
    _check(B.lr_attention_gqa_bwd(q, k, v, heads(o), rows(dout), lse, Bn, S, H, H, 128), want)
    dq, dk, dv = B.lr_attention_bwd(q, heads(k), rows(v), rows(o), heads(dout), lse, Bn, S, H, 128)
    _check([dq, dk, dv], [want[0], heads(want[1]), rows(want[2])])
    _check([B.lr_swiglu_fwd(q, heads(k))], [B.lr_swiglu_fwd(q, k)])
    dg, du = B.lr_swiglu_bwd(q, heads(k), rows(dout))
    want = B.lr_swiglu_bwd(q, k, dout)
    _check([dg, du], [want[0], heads(want[1])])
