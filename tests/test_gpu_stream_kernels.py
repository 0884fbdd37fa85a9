"""GPU parity of the standalone memory-bound kernels against the fp64 oracle."""
import numpy as np
import pytest
import torch

import launches
import synth_inputs as si
from oracle import lowrank_oracle as orc
from parity import check
from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# the last two: enough rows for the backward's row kernel to give a workgroup 128 and 192 rows (its partial
# buffer then has rows that no workgroup owns), the second with a ragged last workgroup
SHAPES = [(1, 8), (37, 72), (300, 1032), (1025, 4096), (32768, 128), (49160, 64)]


@pytest.mark.parametrize("T,d", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rms_stat_apply_bwd(T, d, dtype):
    print(f"rmsnorm kernels T={T} d={d} {dtype}", flush=True)
    eps = 1e-5
    x = si.gaussian(3, "x", (T, d), dtype=dtype)
    gamma = si.gaussian(3, "gamma", (d,), std=0.1, mean=1.0, dtype=dtype)
    dxh = si.gaussian(3, "dxh", (T, d), dtype=dtype)
    dres = si.gaussian(3, "dres", (T, d), dtype=dtype)
    xd, gd, dxhd, dresd = (t.to(DEV) for t in (x, gamma, dxh, dres))
    stat = B.lr_rms_stat(xd)
    xh = B.lr_rmsnorm_apply(xd, gd, stat, eps)
    dx, part = B.lr_rmsnorm_bwd(xd, gd, stat, eps, dxhd, dresd)
    dx2, _ = B.lr_rmsnorm_bwd(xd, gd, stat, eps, dxhd, None)
    torch.cuda.synchronize()
    X, GAM, DXH, DRES = si.f64(x), si.f64(gamma), si.f64(dxh), si.f64(dres)
    check("stat", stat, orc.rms_stat(X), torch.float32, scale=10)
    check("xhat", xh, orc.rmsnorm_fwd(X, GAM, eps)[0], dtype)
    dx_ref, dg_ref = orc.rmsnorm_bwd(X, GAM, eps, DXH)
    check("dx+dres", dx, dx_ref + DRES, dtype)
    check("dx", dx2, dx_ref, dtype)
    check("dgamma", part.sum(0), dg_ref, torch.float32, scale=10)


@pytest.mark.parametrize("T,f", [(5, 16), (129, 344), (2048, 5504)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_act_and_swiglu(T, f, dtype):
    print(f"swiglu kernels T={T} f={f} {dtype}", flush=True)
    g = si.gaussian(4, "g", (T, f), std=2.0, dtype=dtype)
    u = si.gaussian(4, "u", (T, f), dtype=dtype)
    dm = si.gaussian(4, "dm", (T, f), dtype=dtype)
    gd, ud, dmd = (t.to(DEV) for t in (g, u, dm))
    a = B.lr_act_fwd(gd, B.LR_ACT_SILU)
    m = B.lr_swiglu_fwd(gd, ud)
    dg, du = B.lr_swiglu_bwd(gd, ud, dmd)
    torch.cuda.synchronize()
    Gm, U, DM = si.f64(g), si.f64(u), si.f64(dm)
    check("silu", a, orc.silu(Gm), dtype)
    check("m", m, orc.silu(Gm) * U, dtype)
    check("dg", dg, DM * U * orc.silu_prime(Gm), dtype)
    check("du", du, DM * orc.silu(Gm), dtype)


@pytest.mark.parametrize("d", [504, 520, 1024, 1032, 1536, 1544, 2048, 2056, 3072, 3080, 4096])
@pytest.mark.parametrize("T", [3, 69, 449])
def test_rms_bwd_widths(T, d):
    """Both sides of every width at which the row kernel holds another number of slices, on strided rows.  T = 3: no second
    row for any wavefront; 69 and 449: rows that end within a workgroup and within a pair of rows."""
    print(f"rmsnorm backward T={T} d={d}", flush=True)
    eps = 1e-5
    x = si.gaussian(7, "x", (T, d + 8), dtype=torch.bfloat16)[:, :d]
    gamma = si.gaussian(7, "gamma", (d,), std=0.1, mean=1.0, dtype=torch.bfloat16)
    dxh = si.gaussian(7, "dxh", (T, d + 16), dtype=torch.bfloat16)[:, :d]
    dres = si.gaussian(7, "dres", (T, d), dtype=torch.bfloat16)
    big = [torch.full((T, w), float("nan"), dtype=torch.bfloat16, device=DEV) for w in (d + 8, d + 16)]
    big[0][:, :d], big[1][:, :d] = x.to(DEV), dxh.to(DEV)
    xd, dxhd, gd, dresd = big[0][:, :d], big[1][:, :d], gamma.to(DEV), dres.to(DEV)
    stat = B.lr_rms_stat(xd)
    dx = torch.empty((T, d), dtype=torch.bfloat16, device=DEV)
    part = torch.empty((B.lib().lr_rmsnorm_bwd_parts(T), d), device=DEV)
    assert B.lib().lr_rmsnorm_bwd(xd.data_ptr(), d + 8, gd.data_ptr(), stat.data_ptr(), eps, dxhd.data_ptr(), d + 16,
                                  dresd.data_ptr(), d, dx.data_ptr(), d, part.data_ptr(), T, d, B.LR_BF16,
                                  torch.cuda.current_stream().cuda_stream) == 0
    dx_ref, dg_ref = orc.rmsnorm_bwd(si.f64(x), si.f64(gamma), eps, si.f64(dxh))
    check("dx+dres", dx, dx_ref + si.f64(dres), torch.bfloat16)
    check("dgamma", part.sum(0), dg_ref, torch.float32, scale=10)


@pytest.mark.parametrize("T", [16320, 16321, 16448])
def test_rms_bwd_rows_do_not_depend_on_their_number(T):
    """From 256 workgroups on a row of more than 3072 columns is no longer fetched ahead: its results are the same bits."""
    eps, d, n = 1e-5, 3080, 200
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    x, dxh, dres = (torch.randn((T, d), generator=g, device=DEV).bfloat16() for _ in range(3))
    gamma = torch.randn((d,), generator=g, device=DEV).bfloat16()
    stat = B.lr_rms_stat(x)
    dx, part = B.lr_rmsnorm_bwd(x, gamma, stat, eps, dxh, dres)
    for rows in (slice(0, n), slice(T - n, T)):
        few, _ = B.lr_rmsnorm_bwd(x[rows], gamma, stat[rows], eps, dxh[rows], dres[rows])
        assert torch.equal(dx[rows].view(torch.int16), few.view(torch.int16))
    halves = [B.lr_rmsnorm_bwd(x[r], gamma, stat[r], eps, dxh[r], dres[r])[1].sum(0, dtype=torch.float64)
              for r in (slice(0, T // 2), slice(T // 2, T))]
    whole = part.sum(0, dtype=torch.float64)
    # fp32 partials of at most 16 rows per wavefront, each term below max|dxh * n|: a sum of T terms in another order
    assert (whole - halves[0] - halves[1]).abs().max() <= 2 * 20 * 2.0 ** -24 * T * 25


def test_rms_bwd_wide_rows_one_at_a_time_where_there_are_few():
    """More than 3072 columns: the next row is fetched ahead between 16 and 255 workgroups of 64 rows, and rows have the same bits on
    either side of both ends."""
    eps, d = 1e-5, 3080
    g = torch.Generator(device=DEV).manual_seed(6)
    x, dxh, dres = (torch.randn((961, d), generator=g, device=DEV).bfloat16() for _ in range(3))
    gamma = torch.randn((d,), generator=g, device=DEV).bfloat16()
    stat = B.lr_rms_stat(x)

    def kernel(T):
        big = torch.zeros((T, d), dtype=torch.bfloat16, device=DEV)
        return launches.functions(lambda: B.lr_rmsnorm_bwd(big, gamma, torch.ones(T, device=DEV), eps, big, big))[-1]

    kinds = {T: kernel(T) for T in (1, 960, 961, 16320, 16321)}
    assert kinds[1] == kinds[960] == kinds[16321] != kinds[961] == kinds[16320]
    dx, part = B.lr_rmsnorm_bwd(x, gamma, stat, eps, dxh, dres)
    few, fpart = B.lr_rmsnorm_bwd(x[:960], gamma, stat[:960], eps, dxh[:960], dres[:960])
    assert torch.equal(dx[:960].view(torch.int16), few.view(torch.int16))
    last, lpart = B.lr_rmsnorm_bwd(x[960:], gamma, stat[960:], eps, dxh[960:], dres[960:])
    assert torch.equal(dx[960:].view(torch.int16), last.view(torch.int16))
    # the gamma gradient: fp32 partials of the same terms in another order
    whole, parts = part.sum(0, dtype=torch.float64), fpart.sum(0, dtype=torch.float64) + lpart.sum(0, dtype=torch.float64)
    n = x.double() * torch.rsqrt(stat.double() / d + eps)[:, None]
    assert ((whole - parts).abs() <= 2 * 961 * 2.0 ** -24 * (n * dxh.double()).abs().sum(0)).all()
