"""Relative error of CSR A (nmf_csr_relerr) where the residual kernel's runs of
stored entries and its 64-row windows meet the rows in every way: few long
rows, a hub row among short ones, empty rows in front, behind and by the
hundred, rows of one entry, and column ids and values past rowptr[m], which
belong to no row; against the same sums in float64."""
import math

import numpy as np
import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import step

pytestmark = pytest.mark.gpu

LENGTHS = {
    "one entry": [1],
    "two rows": [70001, 3],
    "hub": [2] * 300 + [150000] + [5] * 700,
    "empty ends": [0] * 130 + [7, 0, 0, 64, 65] + [0] * 200 + [1000] + [0] * 70,
    "single entries": [1] * 3000,
    "none": [0] * 10,
    "even": [40] * 5000,
}


@pytest.mark.parametrize("k", [11, 30, 50, 100])
@pytest.mark.parametrize("name", sorted(LENGTHS))
def test_relerr(name, k):
    n, extra = 200000, 37
    length = np.array(LENGTHS[name])
    step("csr relerr %s k=%d" % (name, k))
    rp = np.concatenate([[0], np.cumsum(length)])
    rng = np.random.default_rng(k + len(length))
    ci = np.concatenate([np.sort(rng.choice(n, c, replace=False)) for c in length]
                        + [rng.integers(0, n, extra)]).astype(np.int32)
    v = (rng.random(ci.size) + 1e-3).astype(np.float32)
    m = len(length)
    W, Ht = (torch.from_numpy(rng.random((r, k)).astype(np.float32)).cuda() for r in (m, n))
    got = nmf.nmf_csr_relerr(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(),
                             torch.from_numpy(v).cuda(), n, W, Ht)
    # ||A|| is over the stored values as given
    nnz = int(rp[-1])
    rows = torch.from_numpy(np.repeat(np.arange(m), length)).cuda()
    cols = torch.from_numpy(ci[:nnz].astype(np.int64)).cuda()
    a = torch.from_numpy(v[:nnz]).cuda().double()
    Wd, Hd = W.double(), Ht.double()
    num = float(((Wd.T @ Wd) * (Hd.T @ Hd)).sum())
    if nnz:
        wh = torch.cat([(Wd[rows[p:p + 65536]] * Hd[cols[p:p + 65536]]).sum(1)
                        for p in range(0, nnz, 65536)])
        num += float(((a - wh) ** 2 - wh * wh).sum())
    want = math.sqrt(num / float((torch.from_numpy(v).double() ** 2).sum()))
    # float dot products of k terms, the rest in double
    assert abs(got - want) <= (k + 8) * 2.0 ** -24 * want
