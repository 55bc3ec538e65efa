"""Float products with more terms than 32 slabs of 8192 hold, on nonnegative
data, where an accumulator that cuts bits off is off in one direction and by
more the longer its slab: the relative error of 8192 terms in the 2-norm, 5 u
(u = 2^-24) as stated with the launch shapes, has to hold at any length. Signed
data would hide it."""
import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import U32, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("rows,terms,k", [(70, 2000003, 33), (64, 2200000, 50), (130, 1100000, 64),
                                          (300, 500001, 16), (70, 2000003, 80)])
def test_long_sums(rows, terms, k, trans):
    step("split product of %d terms, %d rows, k=%d trans=%s" % (terms, rows, k, trans))
    g = torch.Generator(device="cuda").manual_seed(terms + k)
    A = torch.rand((terms, rows) if trans else (rows, terms), generator=g, device="cuda")
    F = torch.rand(terms, k, generator=g, device="cuda")
    got = (nmf.nmf_dense_AtF if trans else nmf.nmf_dense_AF)(A, F).double()
    ref = 0
    for r in range(0, terms, 1 << 18):
        B = (A[r:r + (1 << 18)].T if trans else A[:, r:r + (1 << 18)]).double()
        ref = ref + B @ F[r:r + (1 << 18)].double()
    assert float((got - ref).norm() / ref.norm()) <= 8 * U32
