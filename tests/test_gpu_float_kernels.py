"""The float mode's matrix-core kernels at the edges of their tiles, against the CPU checker's definitions."""
import numpy as np
import pytest
import torch

from paper_2502_19913_amd import binding as sp
from paper_2502_19913_amd import synth
from tests.gpuharness import maxerr, relerr

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


# A float sum of K products of unit normals carries a relative rounding error of about sqrt(K) 2^-24 or less: 2e-6 at
# K = 1100.  The bounds allow ten times that over the tensor, and over the largest entry.
PRODUCTS = [  # M, N, K: 32-tiles and one entry; remainders in every dimension that are no multiple of 4 (element-wise
    # access); 64-tiles; 128-tiles; a reduction of one step, of one group past a step, and of several shares (op 2)
    (1, 1, 1), (33, 31, 17), (70, 50, 35), (130, 66, 300), (1100, 515, 33), (1030, 1100, 515), (2048, 2052, 36),
    (2049, 2047, 65), (516, 260, 1100), (36, 68, 4100),
]


@pytest.mark.parametrize("M,N,K", PRODUCTS)
def test_float_products(M, N, K):
    a = synth.normal(41, f"fa{M}{N}{K}", (M, K)); b = synth.normal(42, f"fb{M}{N}{K}", (N, K)); r = synth.normal(43, f"fr{M}{N}{K}", (M, N))
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    guard = 64
    buf = torch.full((M * N + guard,), 7.0, device="cuda")      # entries past the product must stay as they were
    c = buf[:M * N].view(M, N)
    for op, want in ((0, ref + r), (1, ref), (2, ref + 7.0)):
        buf.fill_(7.0)
        if op == 0:
            sp.gemm(0, dev(a), dev(b), c, dev(r))
        elif op == 1:
            sp.gemm(1, dev(a), dev(b.T), c)
        else:
            sp.gemm(2, dev(a.T), dev(b.T), c)
        got = c.cpu().numpy()
        assert relerr(got, want) < 2e-5 and maxerr(got, want) < 2e-5, (op, relerr(got, want), maxerr(got, want))
        assert torch.all(buf[M * N:] == 7.0), op
