"""The float kernels that split their operands into bfloat16 values (products,
residual, rank update) keep float accuracy at any scale of either operand: the
factor or A near the smallest floats while the other side brings the results
back to ordinary size, entries of both sizes in one row, and subnormal
entries. The bars are those of ordinary values, since a power of two on either
operand changes no rounding of an exact split."""
import math

import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import U32, step

pytestmark = pytest.mark.gpu

# (exponent of A, exponent of F): results from 2^-120 to 2^60
SCALES = [(40, -122), (-122, 40), (60, -126), (-100, -20), (100, -126), (0, -125), (-125, 0),
          (30, 30), (64, -60)]


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("m,n,k", [(200, 300, 24), (11590, 11590, 50)])
@pytest.mark.parametrize("ea,ef", SCALES)
def test_product(ea, ef, m, n, k, trans):
    step("split product 2^%d 2^%d %dx%d trans=%s" % (ea, ef, m, n, trans))
    g = torch.Generator(device="cuda").manual_seed(60 + ea)
    A = (torch.rand(m, n, generator=g, device="cuda") + 0.5) * 2.0 ** ea
    F = (torch.rand(m if trans else n, k, generator=g, device="cuda") + 0.5) * 2.0 ** ef
    got = (nmf.nmf_dense_AtF if trans else nmf.nmf_dense_AF)(A, F).double()
    ref = (A.T if trans else A).double() @ F.double()
    rel = (got - ref).abs() / ref
    # positive terms: the mean error of a float sum in slabs, and no entry
    # further off than a truncating accumulation of eight steps' terms
    assert float(rel.norm() / rel.numel() ** 0.5) < 8 * U32
    assert float(rel.max()) <= 2 * 256 * U32


@pytest.mark.parametrize("trans", [False, True])
def test_product_of_mixed_sizes(trans):
    """Rows of A with one entry of ordinary size, at which the factor is zero,
    among entries of 2^-118 at which it is large; subnormal entries."""
    step("split product mixed sizes trans=%s" % trans)
    g = torch.Generator(device="cuda").manual_seed(61)
    A = (torch.rand(128, 320, generator=g, device="cuda") + 0.5) * 2.0 ** -118
    F = (torch.rand(320, 20, generator=g, device="cuda") + 0.5) * 2.0 ** 50
    A[:, 7] = 1.0
    F[7] = 0.0
    F[40:50] = 0.0
    A[:, 40:50] = torch.rand(128, 10, generator=g, device="cuda")
    A[:, 100] = 2.0 ** -149 * torch.randint(1, 1 << 22, (128,), generator=g, device="cuda")
    got = (nmf.nmf_dense_AtF(A.T.contiguous(), F) if trans else nmf.nmf_dense_AF(A, F)).double()
    ref = A.double() @ F.double()
    assert float(((got - ref).abs() / ref).max()) <= 64 * U32


def test_product_of_subnormals():
    """One subnormal entry in each row: the products are exact."""
    step("split product subnormals")
    A = torch.zeros(64, 64, device="cuda")
    bits = torch.arange(1, 65, device="cuda") * 131071 % (1 << 23)
    A[torch.arange(64), torch.arange(64)] = (bits.double() * 2.0 ** -149).float()
    F = torch.full((64, 5), 2.0 ** 100, device="cuda")
    assert torch.equal(nmf.nmf_dense_AF(A, F).double(), (A.double() @ F.double()))
    assert torch.equal(nmf.nmf_dense_AF(F.T.contiguous(), A).double(), F.double().T @ A.double())


@pytest.mark.parametrize("m,n,k", [(100, 200, 20), (700, 1001, 90), (4100, 64, 50)])
@pytest.mark.parametrize("ew,eh", [(0, -118), (-118, 0), (30, -126), (-60, -60), (40, -122)])
def test_residual(m, n, k, ew, eh):
    """A close to W H: the error is 2^-12 of A, far below what a lost third
    plane (2^-16 of W H) would put in its place."""
    step("relerr 2^%d 2^%d %dx%d" % (ew, eh, m, n))
    g = torch.Generator(device="cuda").manual_seed(62)
    W = (torch.rand(m, k, generator=g, device="cuda") + 0.5) * 2.0 ** ew
    Ht = (torch.rand(n, k, generator=g, device="cuda") + 0.5) * 2.0 ** eh
    P = W.double() @ Ht.double().T
    A = (P * (1 + 2.0 ** -12 * torch.rand(m, n, generator=g, device="cuda"))).float()
    got = nmf.nmf_dense_relerr(A, W, Ht)
    na = float(A.double().norm())
    want = float((A.double() - P).norm()) / na
    assert math.isfinite(got)
    # each entry of W H carries at most k + 8 roundings of its terms
    assert abs(got - want) <= (k + 8) * U32 * float(P.norm()) / na


@pytest.mark.parametrize("m,n,k", [(130, 257, 20), (64, 300, 64)])
@pytest.mark.parametrize("e", [-32, -36])
def test_rank_update(m, n, k, e):
    """dL/dA from dL/dP near 2^-120 times H near 2^34, against the same with an
    incoming gradient of ordinary size: linear in it, and dL/dP stays normal
    but for entries below 2^-6 of the others, so the same bits scaled."""
    step("rank update gradients 2^%d" % e)
    g = torch.Generator(device="cuda").manual_seed(63)
    A = (torch.rand(m, n, generator=g, device="cuda") + 0.5) * 2.0 ** 40
    W = torch.rand(m, k, generator=g, device="cuda") + 0.5
    H = (torch.rand(k, n, generator=g, device="cuda") + 0.5) * 2.0 ** 34
    gW = torch.rand(m, k, generator=g, device="cuda") + 0.5
    zero = torch.zeros(k, n, device="cuda")
    _, _, ck = nmf.nmf_hals_unrolled_forward(A, W, H, 1, ckpt_every=1)
    one, _, _ = nmf.nmf_hals_unrolled_backward(A, ck, gW, zero, 1, ckpt_every=1)
    s, _, _ = nmf.nmf_hals_unrolled_backward(A, ck, gW * 2.0 ** e, zero, 1, ckpt_every=1)
    d = (s.double() * 2.0 ** -e - one.double()).norm()
    assert float(d) <= 2.0 ** -22 * float(one.double().norm())
