"""A double product with more than 2^32 outputs: 70,000,001 x 8 at k = 64 is
formed in one slab that the ordered sum copies to the caller's array, over
4.5e9 entries where a dispatch counts its work-items in 32 bits. Every row is
compared with torch's product of its block."""
import pytest

import paper_1609_09154_amd as nmf
from tests.gpu_util import step

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

M, N, K = 70_000_001, 8, 64


def test_every_row_of_a_double_product():
    import torch

    assert M * K > 1 << 32
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(64)
    A = torch.rand((M, N), generator=gen, device=dev, dtype=torch.float64)
    F = torch.rand((N, K), generator=gen, device=dev, dtype=torch.float64)
    ctx = nmf.Context()   # its 36 GB workspace goes with it
    step("double product %d x %d, k = %d" % (M, N, K))
    P = nmf.nmf_dense_AF(A, F, ctx=ctx)
    torch.cuda.synchronize()
    ctx.close()
    worst = 0.0
    for r in range(0, M, 1 << 22):
        worst = max(worst, float((P[r:r + (1 << 22)] - A[r:r + (1 << 22)] @ F).abs().max()))
    del A, F, P
    torch.cuda.empty_cache()
    # sums of 8 terms below 1
    assert worst <= 64 * 2.0 ** -52
