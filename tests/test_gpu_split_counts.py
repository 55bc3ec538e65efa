"""Products whose slab count is chosen to fill the last round of workgroups
(counts that are no power of two), and FP8 A^T W with eight columns a lane (from
2^28 entries of A and 512 columns on), each format and direction, against a double
product of the same stored entries."""
import numpy as np
import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import U32, U64, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,m,n,k", [("f32", 8191, 6007, 100), ("f32", 16700, 9001, 50),
                                      ("f64", 9000, 7000, 20), ("f64", 6007, 8191, 100),
                                      ("bf16", 16400, 9000, 50), ("fp8", 16400, 9008, 20),
                                      ("fp8", 16400, 16416, 20), ("fp8", 32783, 8208, 80),
                                      ("fp8", 524301, 512, 33)])
def test_balanced_slab_counts(dt, m, n, k):
    gen = torch.Generator(device="cuda").manual_seed(m + n + k)
    fd = torch.float64 if dt == "f64" else torch.float32
    # factor entries that every format holds exactly, in one binade per column
    W, Ht = (1 + torch.randint(0, 8, (r, k), generator=gen, device="cuda").to(fd) / 8
             for r in (m, n))
    A = 1 + torch.rand(m, n, generator=gen, device="cuda", dtype=fd)
    A = A.to({"bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}.get(dt, fd))
    u = U64 if dt == "f64" else U32
    for trans, F, K in ((False, Ht, n), (True, W, m)):
        step("balanced slabs %s %dx%d k=%d trans=%s" % (dt, m, n, k, trans))
        got = (nmf.nmf_dense_AtF if trans else nmf.nmf_dense_AF)(A, F)
        X = A.to(torch.float64)
        ref = (X.T.contiguous() if trans else X) @ F.to(torch.float64)
        # nonnegative terms: any order of K rounded additions (and, float, the
        # split's terms) stays within (K + 4) u of the sum
        assert bool(((got.to(torch.float64) - ref).abs() <= (K + 4) * u * ref).all())
        del X, ref
