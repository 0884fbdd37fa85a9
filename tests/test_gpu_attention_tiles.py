"""Causal attention at the edges of its tiles: 32 queries per wavefront, 64 keys per tile, 128 or 256 queries per block."""
import pytest
import torch

import bf16_model as M
import launches
import synth_inputs as si
from oracle import gqa_oracle as gqa
from parity import check
from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HD = 128


@pytest.mark.parametrize("S", [1, 31, 32, 33, 63, 64, 65, 97, 127, 128, 129, 191, 193, 255, 256, 257, 321, 385, 513])
def test_attention_fwd_edges(S):
    """Query blocks in pairs (256 heads in a launch, from 129 tokens on) and a workgroup each (16 heads at a time) give the same bits, and
    those of one batch element lie within the roundings of p and o of the result in 64 bits.  bf16 keeps 8 significant bits, so
    rounding to nearest is off by up to 2^-8 of a value: 2^-8 sum p |v| for the probabilities and 2^-8 |o| <= 2^-8 sum p |v| for
    the output, and 2 % of that for the fp32 arithmetic between."""
    Bn, H, Hkv = 16, 16, 4
    print(f"attention edges S={S}", flush=True)
    g = torch.Generator().manual_seed(S)
    q = torch.randn(Bn * S, H * HD, generator=g).bfloat16()
    k, v = (torch.randn(Bn * S, Hkv * HD, generator=g).bfloat16() for _ in range(2))
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    o, lse = B.lr_attention_gqa_fwd(qd, kd, vd, Bn, S, H, Hkv, HD)
    for b in (0, 7, Bn - 1):
        r = slice(b * S, (b + 1) * S)
        o1, lse1 = B.lr_attention_gqa_fwd(qd[r], kd[r], vd[r], 1, S, H, Hkv, HD)
        assert torch.equal(o[r], o1) and torch.equal(lse.reshape(Bn, -1)[b], lse1.reshape(-1))
    q64 = q[:S].double().view(S, H, HD).transpose(0, 1)
    k64, v64 = (t[:S].double().view(S, Hkv, HD).repeat_interleave(H // Hkv, 1).transpose(0, 1).contiguous() for t in (k, v))
    s = (q64[:, :, None, :] * k64[:, None, :, :]).sum(-1) if S <= 2 else q64 @ k64.transpose(1, 2).contiguous()
    s = (s / HD ** 0.5).masked_fill(torch.ones(S, S, dtype=torch.bool).triu(1), -torch.inf)
    p = s.softmax(-1)
    bound = 2.0 ** -7 * 1.02 * (p @ v64.abs())
    got = o[:S].cpu().double().view(S, H, HD).transpose(0, 1)
    worst = ((got - p @ v64).abs() / bound).max().item()
    assert worst <= 1.0
    assert (lse.view(Bn, H, S)[0].cpu().double() - s.logsumexp(-1)).abs().max() < 1e-4


@pytest.mark.parametrize("S", [65, 129, 255, 257, 513])
def test_attention_bwd_does_not_depend_on_the_launch(S):
    """1, 26 and 64 batch elements of 4 heads (a sequence length that keeps no score gradient).  At 257 tokens that is query blocks of
    128 with a workgroup each, of 256 with a workgroup each, and of 256 in pairs; every form of every length:
    test_attention_bwd_forms."""
    H, Hkv, Bn = 4, 2, 64
    print(f"attention backward launches S={S}", flush=True)
    g = torch.Generator().manual_seed(S)
    q, do = (torch.randn(Bn * S, H * HD, generator=g).bfloat16().to(DEV) for _ in range(2))
    k, v = (torch.randn(Bn * S, Hkv * HD, generator=g).bfloat16().to(DEV) for _ in range(2))
    o, lse = B.lr_attention_gqa_fwd(q, k, v, Bn, S, H, Hkv, HD)
    full = B.lr_attention_gqa_bwd(q, k, v, o, do, lse, Bn, S, H, Hkv, HD)
    for n in (1, 26):
        t = n * S
        part = B.lr_attention_gqa_bwd(q[:t], k[:t], v[:t], o[:t], do[:t], lse[:n].contiguous(), n, S, H, Hkv, HD)
        torch.cuda.synchronize()
        for a, b in zip(part, full):
            assert torch.equal(a, b[:t])


@pytest.mark.parametrize("S", [767, 769, 801, 833, 897, 1027, 1281])
def test_attention_bwd_long(S):
    """The pipelined dK / dV kernel from 768 tokens on, and the other one just below, against the oracle: one to seven tiles in
    its loop, tails of 1 to 63 queries, key blocks of every remainder.  Tolerances as in test_gpu_attention.py."""
    H, Hkv = 2, 1
    print(f"attention backward S={S}", flush=True)
    dt = torch.bfloat16
    q, do = (si.gaussian(17, n, (S, H * HD), dtype=dt) for n in ("q", "do"))
    k, v = (si.gaussian(17, n, (S, Hkv * HD), dtype=dt) for n in ("k", "v"))
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    o, lse = B.lr_attention_gqa_fwd(qd, kd, vd, 1, S, H, Hkv, HD)
    got = B.lr_attention_gqa_bwd(qd, kd, vd, o, dod, lse, 1, S, H, Hkv, HD)
    torch.cuda.synchronize()
    Q, K, V, DO = (si.f64(t) for t in (q, k, v, do))
    o_ref, _ = gqa.attention_gqa_fwd(Q, K, V, 1, S, H, Hkv, HD)
    refs = gqa.attention_gqa_bwd(Q, K, V, DO, 1, S, H, Hkv, HD)
    bud = M.attention_budget(Q, K, V, DO, 1, S, H, Hkv, HD, o_ref, *refs)
    for n, a, r in zip(("dq", "dk", "dv"), got, refs):
        check(n, a, r, dt, bud[n])


@pytest.mark.parametrize("S,Bn,H,threads", [(16, 24, 16, 256), (64, 24, 16, 256), (200, 24, 16, 256), (320, 24, 16, 256), (1024, 4, 32, 256),
                                            (1793, 2, 32, 512), (2047, 2, 32, 512), (2047, 4, 32, 256), (2049, 2, 32, 256),
                                            (3584, 1, 32, 512)])
def test_attention_fwd_width_of_a_block(S, Bn, H, threads):
    """Blocks of 128 queries, and of 256 where a launch is one pair of those for each CU, from eight blocks on: elsewhere wide
    blocks leave wavefronts waiting."""
    print(f"attention forward launch S={S}", flush=True)
    q = torch.zeros((Bn * S, H * HD), dtype=torch.bfloat16, device=DEV)
    blocks = -(-S // (threads // 2))
    per_wg = 1 if blocks * Bn * H <= 256 else 2
    assert launches.of(lambda: B.lr_attention_fwd(q, q, q, Bn, S, H, HD)) == [(-(-blocks // per_wg) * Bn * H, threads, 65536)]


@pytest.mark.parametrize("S", [1793, 1825, 1983, 2015, 2047, 2048, 2049, 2111, 2304])
def test_attention_fwd_long(S):
    """Sequences of more blocks than test_attention_fwd_edges has: blocks of 256 queries up to 2048 tokens, pairs of blocks of 128 beyond
    (64 heads), and a workgroup for each block of 128 (4 heads); on one head against 64 bits, bounds as there."""
    Bn, H = 8, 8
    print(f"attention forward S={S}", flush=True)
    g = torch.Generator().manual_seed(S)
    q, k, v = (torch.randn(Bn * S, H * HD, generator=g).bfloat16() for _ in range(3))
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    o, lse = B.lr_attention_fwd(qd, kd, vd, Bn, S, H, HD)
    for b in (0, Bn - 1):
        r = slice(b * S, (b + 1) * S)
        part = [t[r, 4 * HD:].contiguous() for t in (qd, kd, vd)]
        o1, lse1 = B.lr_attention_fwd(*part, 1, S, 4, HD)
        assert torch.equal(o[r, 4 * HD:], o1) and torch.equal(lse.view(Bn, H, S)[b, 4:], lse1.view(4, S))
    q64, k64, v64 = (t[:S, :HD].double() for t in (q, k, v))
    s = (q64 @ k64.t() / HD ** 0.5).masked_fill(torch.ones(S, S, dtype=torch.bool).triu(1), -torch.inf)
    p = s.softmax(-1)
    assert ((o[:S, :HD].cpu().double() - p @ v64).abs() <= 2.0 ** -7 * 1.02 * (p @ v64.abs())).all()
    assert (lse.view(Bn, H, S)[0, 0].cpu().double() - s.logsumexp(-1)).abs().max() < 1e-4


def _bwd_launches(S, n, H, Hkv):
    """dQ and dK / dV of a backward over n sequences: (workgroups, threads, LDS) of both"""
    q, k = (torch.zeros((n * S, h * HD), dtype=torch.bfloat16, device=DEV) for h in (H, Hkv))
    lse = torch.zeros((n, H, S), device=DEV)
    return launches.of(lambda: B.lr_attention_gqa_bwd(q, k, k, q, q, lse, n, S, H, Hkv, HD))[1:3]


def _compare_parts(S, n, parts, H, Hkv):
    g = torch.Generator().manual_seed(S)
    q, do = (torch.randn(n * S, H * HD, generator=g).bfloat16().to(DEV) for _ in range(2))
    k, v = (torch.randn(n * S, Hkv * HD, generator=g).bfloat16().to(DEV) for _ in range(2))
    o, lse = B.lr_attention_gqa_fwd(q, k, v, n, S, H, Hkv, HD)
    full = B.lr_attention_gqa_bwd(q, k, v, o, do, lse, n, S, H, Hkv, HD)
    for m in parts:
        r, last = slice((n - m) * S, n * S), slice(n - m, n)     # (the last ones: their blocks are the launch's last)
        part = B.lr_attention_gqa_bwd(q[r], k[r], v[r], o[r], do[r], lse[last].contiguous(), m, S, H, Hkv, HD)
        torch.cuda.synchronize()
        for a, b in zip(part, full):
            assert torch.equal(a, b[r])


@pytest.mark.parametrize("S,batches", [(65, (1, 66)), (129, (1, 40, 66)), (255, (1, 40, 66)), (257, (1, 26, 40)), (513, (1, 16, 30))])
def test_attention_bwd_forms(S, batches):
    """dQ on blocks of 128 queries, on blocks of 256 and on pairs
    of those: batches of 4 heads that take one form each, the same bits from all."""
    H, Hkv = 4, 2
    print(f"attention backward forms S={S} B={batches}", flush=True)
    n128, n256 = (S + 127) // 128, (S + 255) // 256
    grids = [n128 * H * batches[0], *([n256 * H * batches[1]] if len(batches) == 3 else []), (n256 + 1) // 2 * H * batches[-1]]
    assert [_bwd_launches(S, n, H, Hkv)[0][0] for n in batches] == grids
    assert n128 * H * batches[0] <= 256 < n256 * H * batches[-1]
    assert len(batches) == 2 or n256 * H * batches[1] <= 256 < n128 * H * batches[1]
    _compare_parts(S, batches[-1], batches[:-1], H, Hkv)


@pytest.mark.parametrize("S", [769, 897, 1023, 1025, 1087, 1153, 1283])
def test_attention_bwd_paired_key_blocks(S):
    """Launches whose workgroups take two key blocks, the second one with the ring that the first has used: odd and even numbers of
    blocks (an odd one has a middle block without a mirror), from 1024 tokens on with the pipelined kernel.  The bits of one
    sequence, a workgroup per block, which test_attention_bwd_long checks against the oracle."""
    H, Hkv, n = 4, 2, 11
    print(f"attention backward, paired key blocks S={S}", flush=True)
    blocks, long_lds = (S + 127) // 128, 4 * (2 * 64 * 256 + 512) + 256
    many, one = _bwd_launches(S, n, H, Hkv)[1], _bwd_launches(S, 1, H, Hkv)[1]
    assert many[0] == (blocks + 1) // 2 * H * n and one[0] == blocks * H
    assert (many[2] == long_lds) == (S >= 1024) and one[2] == long_lds
    _compare_parts(S, n, (1,), H, Hkv)


@pytest.mark.parametrize("S,n", [(257, 40), (289, 40), (383, 40), (511, 36), (513, 22), (1025, 13), (1283, 12), (1799, 9)])
def test_attention_bwd_pairs_of_wavefronts(S, n):
    """256 keys per workgroup, in pairs of blocks: the bits of the other kernels, which one sequence takes; also of what an infinite
    gradient reaches (the keys that its query sees, and those of its 32 x 32 block)."""
    H, Hkv = 4, 2
    print(f"attention backward, pairs of wavefronts S={S} B={n}", flush=True)
    many, one = _bwd_launches(S, n, H, Hkv)[1], _bwd_launches(S, 1, H, Hkv)[1]
    assert many[:2] == (((S + 255) // 256 + 1) // 2 * H * n, 512) and one[1] == 256
    _compare_parts(S, n, (1,), H, Hkv)
    g = torch.Generator().manual_seed(S)
    q, do = (torch.randn(n * S, H * HD, generator=g).bfloat16().to(DEV) for _ in range(2))
    k, v = (torch.randn(n * S, Hkv * HD, generator=g).bfloat16().to(DEV) for _ in range(2))
    do[torch.tensor([5, 70, S - 1]) - S, torch.tensor([3, HD + 9, 3 * HD])] = torch.inf    # a query of three heads of the last sequence
    o, lse = B.lr_attention_gqa_fwd(q, k, v, n, S, H, Hkv, HD)
    full = B.lr_attention_gqa_bwd(q, k, v, o, do, lse, n, S, H, Hkv, HD)
    part = B.lr_attention_gqa_bwd(*(t[-S:] for t in (q, k, v, o, do)), lse[n - 1:].contiguous(), 1, S, H, Hkv, HD)
    for a, b in zip(part, full):
        assert a.isnan().any() and torch.equal(a.nan_to_num(nan=7.0), b[-S:].nan_to_num(nan=7.0))


@pytest.mark.parametrize("S,n", [(1025, 10), (1281, 9), (2047, 6)])
def test_attention_bwd_paired_query_blocks(S, n):
    """dQ on blocks of 128 queries and their mirrors, where blocks of 256 are no more than CUs: odd and even numbers of blocks; the
    bits of one sequence, a workgroup per block."""
    H, Hkv = 4, 2
    print(f"attention backward, paired query blocks S={S} B={n}", flush=True)
    n128, n256 = (S + 127) // 128, (S + 255) // 256
    assert n256 * H * n <= 256 < n128 * H * n
    assert [_bwd_launches(S, m, H, Hkv)[0][:2] for m in (n, 1)] == [((n128 + 1) // 2 * H * n, 256), (n128 * H, 256)]
    _compare_parts(S, n, (1,), H, Hkv)


@pytest.mark.parametrize("S,n", [(264, 40), (288, 40), (512, 36), (776, 18), (1280, 13), (2048, 9)])
def test_attention_bwd_score_gradient_kept_or_formed_twice(S, n):
    """Multiples of 8 tokens: one sequence stores the score gradient for dQ's product, enough of them form it twice; the same bits."""
    H, Hkv = 4, 2
    print(f"attention backward, score gradient kept or not S={S} B={n}", flush=True)
    pairs = ((S + 255) // 256 + 1) // 2 * H * n
    many, one = _bwd_launches(S, n, H, Hkv), _bwd_launches(S, 1, H, Hkv)
    assert [k[:2] for k in many] == [(pairs, 512)] * 2 and one[0][:2] == ((S + 127) // 128 * H, 512)
    _compare_parts(S, n, (1,), H, Hkv)


@pytest.mark.parametrize("S,n", [(8, 80), (136, 40), (136, 70), (520, 21), (1536, 10), (1536, 11), (1544, 9), (2056, 7)])
def test_attention_bwd_key_blocks_of_pairs_or_of_wavefronts(S, n):
    """Multiples of 8 tokens whose score gradient is stored: by four pairs of wavefronts where a workgroup has a CU, by four
    wavefronts where it has not; the same bits."""
    H, Hkv = 4, 2
    print(f"attention backward, key blocks S={S} B={n}", flush=True)
    nkb = (S + 127) // 128
    for m in (1, n):
        wide = nkb * H * m <= 256 or (nkb * H * m <= 512 and S <= 1536)
        blocks = (nkb if nkb * H * m <= 256 else (nkb + 1) // 2) * H * m
        assert _bwd_launches(S, m, H, Hkv)[0][:2] == (blocks, 512 if wide else 256)
    _compare_parts(S, n, (1, n // 2), H, Hkv)
