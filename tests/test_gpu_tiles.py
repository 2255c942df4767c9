"""bf16 matrix products at the edges of every tile size, against float64 products of the same bf16 values."""
import numpy as np
import pytest
import torch

from paper_2502_19913_amd import binding as sp
from paper_2502_19913_amd import synth
from tests.gpuharness import maxerr, relerr, round_bf16

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda().bfloat16()


# M, N, K: one 16-byte chunk; one 64-tile less, exactly and one chunk more in every dimension; 64-tiles with steps below,
# at and past the ring's five slots; 128-tiles with remainders past its four slots; 256-tiles with remainders; a reduction
# cut into runs that are no multiple of the ring (op 2, 64-tiles)
PRODUCTS = [
    (8, 8, 8), (56, 56, 56), (64, 64, 64), (72, 72, 72), (72, 136, 320), (200, 72, 1032), (1000, 1032, 136), (1032, 1000, 256),
    (2056, 1160, 328), (4096, 2824, 72), (4000, 1032, 200), (520, 264, 2056),
]
# 128-tiles of three, four and five steps; 64-, 128- and 256-tiles of which a workgroup takes several in turn; op 2 in
# several runs of 128- and 256-tiles.  tests/test_host.py checks against the dispatch that the lists hold what they say.
PRODUCTS += [(1288, 1544, 192), (1288, 1544, 200), (1288, 1544, 264), (6664, 520, 200), (20670, 272, 1472), (8200, 2312, 72),
             (1032, 1032, 3080), (2056, 2056, 2056)]
# R, h, d; the last four: several 64- and 128-tiles in turn, forward and backward
FEED_FORWARD = [(1, 64, 64), (65, 64, 72), (999, 768, 288), (129, 192, 96), (2050, 1408, 512), (4100, 2816, 64),
                (675, 2752, 64), (723, 2752, 64), (6657, 576, 200), (20489, 320, 1480)]


@pytest.mark.parametrize("M,N,K", PRODUCTS)
def test_products_at_tile_edges(M, N, K):
    a = round_bf16(synth.normal(51, f"ta{M}{N}{K}", (M, K))); b = round_bf16(synth.normal(52, f"tb{M}{N}{K}", (N, K)))
    r = round_bf16(synth.normal(53, f"tr{M}{N}{K}", (M, N)))
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    guard = 64
    for op, want in ((0, ref + r), (1, ref), (2, ref + 7.0)):
        buf = torch.full((M * N + guard,), 7.0, device="cuda", dtype=torch.float32 if op == 2 else torch.bfloat16)
        c = buf[:M * N].view(M, N)
        if op == 0:
            sp.gemm(0, dev(a), dev(b), c, dev(r))
        elif op == 1:
            sp.gemm(1, dev(a), dev(b.T), c)
        else:
            sp.gemm(2, dev(a.T), dev(b.T), c)
        got = c.float().cpu().numpy()
        # op 0/1: bf16 roundings of the product and of the sum with R: half a unit in the last of 8 bits, up to 2^-8 of an
        # entry each, and a quarter for products larger than their sum with R; op 2: float sums, about sqrt(K) 2^-24 or
        # less, allowed ten times that at K = 2056
        lim = 3e-5 if op == 2 else 2.25 * 2.0 ** -8
        assert relerr(got, want) < lim and maxerr(got, want) < lim, (op, relerr(got, want), maxerr(got, want))
        assert torch.all(buf[M * N:] == 7.0), op


@pytest.mark.parametrize("R,h,d", FEED_FORWARD)
def test_feed_forward_epilogues_at_tile_edges(R, h, d):
    hn = round_bf16(synth.normal(54, f"th{R}{h}", (R, d))); w = round_bf16(synth.normal(55, f"tw{R}{h}", (2 * h, d)) / np.sqrt(d))
    dy = round_bf16(synth.normal(56, f"ty{R}{h}", (R, d))); wd = round_bf16(synth.normal(57, f"tv{R}{h}", (d, h)) / np.sqrt(d))
    gu = torch.empty(R, 2 * h, device="cuda", dtype=torch.bfloat16); act = torch.empty(R, h, device="cuda", dtype=torch.bfloat16)
    dgu = torch.empty_like(gu); tmp = torch.empty_like(act)
    sp.ffn_up_fwd(dev(hn), dev(w), gu, act)
    sp.ffn_down_bwd(dev(dy), dev(wd), gu, dgu, tmp)
    got = gu.float().cpu().numpy().astype(np.float64)
    g, u = got[:, :h], got[:, h:]
    sg = 1 / (1 + np.exp(-g))
    da = dy.astype(np.float64) @ wd.astype(np.float64)
    # bf16 roundings of up to 2^-8 each: gate|up one; act one; d(gate)|d(up) two (d(act), then the result)
    for name, x, want, n in (("gate|up", got, hn.astype(np.float64) @ w.astype(np.float64).T, 1),
                             ("act", act.float().cpu().numpy(), g * sg * u, 1),
                             ("d(gate)|d(up)", dgu.float().cpu().numpy(),
                              np.concatenate([da * u * sg * (1 + g * (1 - sg)), da * g * sg], 1), 2)):
        lim = (n + 0.25) * 2.0 ** -8
        assert relerr(x, want) < lim and maxerr(x, want) < lim, (name, relerr(x, want), maxerr(x, want))


@pytest.mark.parametrize("M,N,K", [(72, 136, 320), (1288, 1544, 192), (4096, 2824, 72), (2056, 1160, 328)])
def test_a_sum_in_place_has_the_bits_of_one_beside(M, N, K):
    """R may be the output: a thread reads a batch of its own entries of R before it stores them (tiles of every size, the last
    row and column of tiles partly outside the matrix)."""
    a, b = dev(synth.normal(61, f"ia{M}", (M, K))), dev(synth.normal(62, f"ib{M}", (N, K)))
    r = dev(synth.normal(63, f"ir{M}", (M, N)))
    c = torch.empty_like(r)
    sp.gemm(0, a, b, c, r)
    sp.gemm(0, a, b, r, r)
    assert torch.equal(c, r)
