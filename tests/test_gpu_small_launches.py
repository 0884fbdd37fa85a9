"""Short passes that share a launch: the gamma fold beside the row statistic, the finishing pass of a normed weight gradient with its dgamma,
the rotation of queries and keys."""
import pytest
import torch

import launches
from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _group(T, d, r, n, G, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x, dy = (torch.randn(s, generator=g, device=DEV).to(dtype) for s in ((T, d), (G, T, n)))
    wd = (torch.randn((G * r, d), generator=g, device=DEV) * d ** -0.5).to(dtype)
    wu = (torch.randn((G, n, r), generator=g, device=DEV) * r ** -0.5).to(dtype)
    gamma = 2.0 ** torch.randint(-2, 3, (d,), generator=g, device=DEV)       # (divides out of a gradient exactly)
    return x, gamma.to(dtype), wd, wu, dy


# rows of the gradient G r: of one partial of dgamma, one and a remainder, a chunk of 128 rows and its edges, the most that one
# workgroup takes and more; columns short of a strip, of several, the most and more
@pytest.mark.parametrize("d,r,G", [(8, 8, 1), (264, 16, 2), (256, 64, 2), (520, 136, 1), (1016, 64, 3), (1024, 128, 2), (1032, 128, 2), (256, 264, 1)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_dgamma_of_few_rows(d, r, G, dtype):
    T, n = 200, 72
    print(f"dgamma d={d} r={r} G={G} {dtype}", flush=True)
    x, gamma, wd, wu, dy = _group(T, d, r, n, G, dtype, d)
    z, stat, _ = B.lr_group_fwd(x, gamma, 1e-5, B.LR_NORM_ONLINE, wd, wu)
    back = lambda grads=None: B.lr_group_bwd(x, gamma, 1e-5, B.LR_NORM_ONLINE, wd, wu, z, stat, dy, grads=grads)
    _, dg, dwd, dwu = back()
    torch.cuda.synchronize()
    terms = wd.double() * (dwd.double() / gamma.double())
    # (a chain of up to 8 of a class, 4 classes, the partials; each rounding at most 2^-24 of what has been added up)
    bound = (12 + G * r / 32) * 2.0 ** -24 * terms.abs().sum(0)
    assert ((dg.double() - terms.sum(0)).abs() <= bound).all()
    start = [torch.full_like(t, 0.5) for t in (dg, dwd, dwu)]
    more = back([t.clone() for t in start])[1:]
    torch.cuda.synchronize()
    assert torch.equal(more[0], dg + 0.5) and torch.equal(more[1], dwd + 0.5)


# rows and partials on both sides of each line: all of one turn of a workgroup, of two up to 12 partials, of three with one; in fp32, whose
# turns have 8 rows, up to 16 rows, up to 32 with 4 partials
@pytest.mark.parametrize("dtype,rows,T,partials,whole", [
    (torch.bfloat16, 64, 10000, 18, True), (torch.bfloat16, 72, 6144, 12, True), (torch.bfloat16, 128, 6144, 12, True),
    (torch.bfloat16, 72, 6656, 13, False), (torch.bfloat16, 128, 16384, 32, False), (torch.bfloat16, 136, 512, 1, True),
    (torch.bfloat16, 192, 512, 1, True), (torch.bfloat16, 192, 2048, 4, False), (torch.bfloat16, 200, 512, 1, False),
    (torch.float32, 16, 8200, 4, True), (torch.float32, 17, 8200, 4, True), (torch.float32, 32, 512, 1, True),
    (torch.float32, 32, 16400, 8, False), (torch.float32, 33, 512, 1, False), (torch.float32, 192, 512, 1, False)])
def test_one_launch_for_few_rows_and_partials(dtype, rows, T, partials, whole):
    d, n = 136, 72
    print(f"finishing pass {dtype} rows={rows} T={T}", flush=True)
    x, gamma, wd, wu, dy = _group(T, d, rows, n, 1, dtype, rows)
    z, stat, _ = B.lr_group_fwd(x, gamma, 1e-5, B.LR_NORM_ONLINE, wd, wu)
    back = lambda: B.lr_group_bwd(x, gamma, 1e-5, B.LR_NORM_ONLINE, wd, wu, z, stat, dy)
    _, dg, dwd, _ = back()
    torch.cuda.synchronize()
    terms = wd.double() * (dwd.double() / gamma.double())
    assert ((dg.double() - terms.sum(0)).abs() <= (12 + rows / 32) * 2.0 ** -24 * terms.abs().sum(0)).all()      # (as above)
    # (the pass behind the norm comes after the others, which have no dgamma; its second argument is the number of partials)
    name, count = [(name, launches.words(args[1], 1)[0]) for name, args in launches.named(back, "wgrad_finish") if "many" not in name][-1]
    assert (count, "whole" in name) == (partials, whole)


# rows that don't fill a workgroup, and more weight vectors than a workgroup's
@pytest.mark.parametrize("T,d,r,G", [(1, 64, 520, 1), (7, 2056, 264, 2), (1031, 520, 176, 3)])
def test_fold_beside_the_row_statistic(T, d, r, G):
    print(f"fold and statistic T={T} d={d} r={r} G={G}", flush=True)
    x, gamma, wd, wu, _ = _group(T, d, r, 64, G, torch.bfloat16, T)
    run = lambda: B.lr_group_fwd(x, gamma, 1e-5, B.LR_NORM_ONLINE, wd, wu)
    z, stat, _ = run()
    assert torch.equal(stat, B.lr_rms_stat(x))
    assert launches.of(run)[0][0] == (T + 3) // 4 + (G * r * d // 8 + 255) // 256
    # with gamma folded in by hand (powers of two: exact) the same product
    z1 = B.lr_group_fwd(x, torch.ones_like(gamma), 1e-5, B.LR_NORM_ONLINE, wd * gamma, wu)[0]
    torch.cuda.synchronize()
    assert torch.equal(z, z1)
