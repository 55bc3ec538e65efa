"""Float products on the bfloat16 cores (nmf_dense_AF, nmf_dense_AtF): edges of
the kernel's tiles and steps, both launch shapes and the largest ranks against
a float64 product, and the entries for which the three-way split does not
hold (infinities, NaN, values that round to infinity as bfloat16, values
whose last bits fall below the smallest bfloat16)."""
import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import U32, step

pytestmark = pytest.mark.gpu

# rows and columns of A around the 16-row tiles, the 32-value steps and one
# and two columns; k around the 16-column tiles
SHAPES = [(1, 1, 1), (1, 40, 3), (40, 1, 17), (2, 3, 16), (3, 2, 5), (31, 33, 16), (32, 32, 15),
          (33, 31, 1), (129, 255, 48), (257, 64, 65), (64, 1025, 80), (515, 130, 96),
          (1000, 777, 112), (777, 1000, 128), (8200, 2049, 50), (127, 70001, 30)]
# 2^27 entries and up: the wide shape at k <= 64, ragged both ways
WIDE = [(8193, 16400, 50), (16383, 8195, 16), (70, 2000003, 33), (11590, 11590, 100)]


def products(A, F, trans):
    return (nmf.nmf_dense_AtF if trans else nmf.nmf_dense_AF)(A, F)


def check(A, F, trans):
    """|P - A F| against the standard bound of a K-term sum in unit roundoff
    u, K u |A| |F| with the constant 2 (truncating accumulation), and at
    least eight roundings."""
    Ad, Fd = (A.T if trans else A).double(), F.double()
    got = products(A, F, trans).double()
    ref, mag = Ad @ Fd, Ad.abs() @ Fd.abs()
    K = Fd.shape[0]
    err = (got - ref).abs()
    assert got.shape == ref.shape
    assert bool((err <= 2 * max(K, 8) * U32 * mag).all()), float((err / mag).max())
    # far below the worst case: no further than 32 roundings in the mean
    assert float(err.norm() / mag.norm()) < 32 * U32


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("m,n,k", SHAPES + WIDE)
def test_product(m, n, k, trans):
    step("split product %dx%d k=%d trans=%s" % (m, n, k, trans))
    g = torch.Generator(device="cuda").manual_seed(m * 7 + n * 3 + k)
    A = torch.randn(m, n, generator=g, device="cuda")
    F = torch.randn(m if trans else n, k, generator=g, device="cuda")
    check(A, F, trans)


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("m,n,k", [(100, 333, 20), (8193, 16400, 50)])
def test_special_values(m, n, k, trans):
    step("split product specials %dx%d trans=%s" % (m, n, trans))
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.rand(m, n, generator=g, device="cuda")
    F = torch.rand(m if trans else n, k, generator=g, device="cuda") + 0.5
    F[7, 3] = 0.0
    A[3, 7] = float("inf")
    A[50, 60] = 3.4e38 * 0.9999999
    A[90, 9] = float("nan")
    F[11, 5] = float("inf")
    Ad = A.T if trans else A
    got = products(A, F, trans)
    # row by row: a sum with an infinity or a NaN has the value that its terms
    # give in any order; finite sums keep the bound
    ref = (Ad.double() @ F.double()).float()
    assert bool((torch.isnan(got) == torch.isnan(ref)).all())
    assert bool((torch.isinf(got) == torch.isinf(ref)).all())
    fin = torch.isfinite(ref)
    err = (got.double() - ref.double()).abs()[fin]
    assert bool((err <= 2 * F.shape[0] * U32 * ref.double().abs()[fin]).all())


@pytest.mark.parametrize("scale_a,scale_f", [(2.0 ** -118, 1.0), (1.0, 2.0 ** -118),
                                             (2.0 ** -112, 2.0 ** 40)])
def test_small_values(scale_a, scale_f):
    step("split product small values %g %g" % (scale_a, scale_f))
    g = torch.Generator(device="cuda").manual_seed(6)
    for trans in (False, True):
        A = (torch.rand(200, 300, generator=g, device="cuda") + 0.5) * scale_a
        F = (torch.rand(200 if trans else 300, 24, generator=g, device="cuda") + 0.5) * scale_f
        check(A, F, trans)
