"""The gate's and the up product of the MLP in one launch that keeps the gate's tile in registers, where that is estimated to be
faster.  While launches are being timed each product has its own: every output has to have the same bits, with the gate and up
activations kept by the caller or not."""
import pytest
import torch

import launches
import synth_inputs as si
from paper_2512_12131_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# one row to several tiles of each size (32, 64, 64 x 128, 128), remainders of rows, columns and k, one slice of k and an odd number
@pytest.mark.parametrize("T,H,f,r", [(1, 1, 200, 8), (33, 2, 344, 72), (130, 1, 1000, 64), (300, 4, 1003, 136), (777, 8, 2730, 128),
                                     (3000, 4, 1376, 64), (5000, 8, 2752, 168)])
def test_forward_and_backward(T, H, f, r):
    print(f"gate and up in one launch T={T} H={H} f={f} r={r}", flush=True)
    d, f_ld = 128 * H, (f + 7) // 8 * 8
    case = si.block_case(1, T, d, H, 128, f, r, seed=5)
    p = {k: v.to(DEV) for k, v in si.pack_block_params(case["params"], f, f_ld).items()}
    x, dy = case["x"].to(DEV), case["dy"].to(DEV)
    desc = B.make_block_desc(1, T, d, H, 128, f, f_ld, r)
    # gamma folded, three pairs of projections with the attention, the residual's row sums, and gate / up: one launch less
    assert len(launches.of(lambda: B.lr_block_fwd(desc, p, x))) == 11

    def step():
        y, ck = B.lr_block_fwd(desc, p, x)
        dx, grads = B.lr_block_bwd(desc, p, x, dy, ck)
        ys, cks, saved = B.lr_block_fwd_save(desc, p, x)
        return [y, *ck.values(), dx, *grads.values(), ys, *cks.values(), *saved.values()]

    together = step()
    B.lr_launch_timer_begin(400)
    apart = step()
    torch.cuda.synchronize()
    B.lr_launch_timer_end()
    for a, b in zip(together, apart):
        assert torch.equal(a, b)


def test_longest_first_in_a_joint_launch():
    """Beside products whose k lies between its own and twice that, the pair is the one that takes longest: its workgroups start first."""
    T, H, f, r = 128, 1, 344, 120
    print(f"gate and up first in a joint launch T={T} H={H} f={f} r={r}", flush=True)
    d = 128 * H
    case = si.block_case(1, T, d, H, 128, f, r, seed=6)
    p = {k: v.to(DEV) for k, v in si.pack_block_params(case["params"], f, f).items()}
    x, dy = case["x"].to(DEV), case["dy"].to(DEV)
    desc = B.make_block_desc(1, T, d, H, 128, f, f, r)
    y, ck = B.lr_block_fwd(desc, p, x)
    # (a product's sizes M, N, K lie among its first words)
    firsts = [launches.words(args[0], 24)[20:23] for _, args in launches.named(lambda: B.lr_block_bwd(desc, p, x, dy, ck), "gemm_joint_kernel")]
    assert [T, f, r] in firsts
