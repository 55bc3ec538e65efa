"""dL/dA of the unrolled MU layer at the edges of the float rank update's
128 x 128 blocks and 32-entry steps (odd counts of 16-entry units, ragged and
tiny matrices, several passes over a long segment), against the float64
layer's, which another kernel forms."""
import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import U32, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,iters,every", [
    (1, 1, 1, 1, 1), (3, 130, 5, 3, 3), (129, 5, 16, 1, 1), (128, 128, 33, 2, 2),
    (257, 131, 48, 3, 2), (300, 513, 64, 5, 5), (64, 1000, 20, 7, 10), (200, 150, 64, 80, 80)])
def test_gA(m, n, k, iters, every):
    step("rank update %dx%d k=%d T=%d c=%d" % (m, n, k, iters, every))
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    A = torch.rand(m, n, generator=g, device="cuda") + 0.1
    W = torch.rand(m, k, generator=g, device="cuda") + 0.1
    H = torch.rand(k, n, generator=g, device="cuda") + 0.1
    gW = torch.randn(m, k, generator=g, device="cuda")
    gH = torch.randn(k, n, generator=g, device="cuda")
    _, _, ck = nmf.nmf_mu_unrolled_forward(A, W, H, iters, ckpt_every=every)
    gA, _, _ = nmf.nmf_mu_unrolled_backward(A, ck, gW, gH, iters, ckpt_every=every)
    # the same gradient in float64, whose rank update is the other kernel
    _, _, ck = nmf.nmf_mu_unrolled_forward(A.double(), W.double(), H.double(), iters,
                                           ckpt_every=every)
    rA, _, _ = nmf.nmf_mu_unrolled_backward(A.double(), ck, gW.double(), gH.double(), iters,
                                            ckpt_every=every)
    # float32 throughout: each iteration's states and gradients carry a few
    # roundings of K-term sums, compounded over the iterations
    tol = 64 * U32 * (iters + 2) * max(1.0, (m + n) ** 0.5 / 8)
    assert float((gA.double() - rA).norm()) <= tol * float(rA.norm())
