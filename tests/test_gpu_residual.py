"""Relative error of dense A (nmf_dense_relerr) at the edges of the residual
kernel's 16-row and 64-column tiles and of its runs of rows, for every element
type and rank class, against the residual formed in float64."""
import math

import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import U32, U64, step

pytestmark = pytest.mark.gpu

TYPES = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16,
         "fp8": torch.float8_e4m3fn}
# (m, n, k): one entry, tiles of 16 rows and 64 columns and their neighbours,
# runs of rows of every length, each 32-wide rank step
SHAPES = [(1, 16, 1), (15, 64, 16), (17, 48, 17), (64, 128, 32), (65, 80, 33), (1000, 208, 64),
          (333, 4096, 65), (4100, 16, 100), (70, 20000, 128), (9001, 1504, 50), (128, 144, 112)]
RAGGED = [(1, 1, 1), (3, 2, 4), (16, 63, 8), (50, 65, 47), (700, 1001, 90), (2001, 130, 128)]


def check(m, n, k, dt, A, W, Ht, u):
    got = nmf.nmf_dense_relerr(A, W, Ht)
    Ad = A.float().double() if A.dtype != torch.float64 else A
    D = Ad - W.double() @ Ht.double().T
    na = float(Ad.norm())
    want = float(D.norm()) / na
    # each entry of W H carries at most (k + 8) roundings of its terms, the
    # sums of squares are exact to double
    slack = (k + 8) * u * float((W.double().abs() @ Ht.double().abs().T).norm()) / na
    assert math.isfinite(got)
    assert abs(got - want) <= slack + 1e-13 * want, (got, want, slack)


@pytest.mark.parametrize("dt", sorted(TYPES))
@pytest.mark.parametrize("m,n,k", SHAPES + RAGGED)
def test_relerr(dt, m, n, k):
    if dt in ("bf16", "fp8") and n % 16:
        pytest.skip("reduced-precision rows are multiples of 16 bytes")
    step("relerr %s %dx%d k=%d" % (dt, m, n, k))
    g = torch.Generator(device="cuda").manual_seed(m + 3 * n + 5 * k)
    fdt = torch.float64 if dt == "f64" else torch.float32
    W = torch.rand(m, k, generator=g, device="cuda", dtype=fdt)
    Ht = torch.rand(n, k, generator=g, device="cuda", dtype=fdt)
    A = W @ Ht.T + 0.1 * torch.rand(m, n, generator=g, device="cuda", dtype=fdt)
    check(m, n, k, dt, A.to(TYPES[dt]), W, Ht, U64 if dt == "f64" else U32)


def test_relerr_of_infinite_product():
    """A product past the largest float is an infinite error, not a NaN."""
    step("relerr infinite product")
    A = torch.rand(100, 200, device="cuda")
    W = torch.rand(100, 20, device="cuda") + 0.5
    Ht = torch.rand(200, 20, device="cuda") + 0.5
    W[3] = 3e38
    assert nmf.nmf_dense_relerr(A, W, Ht) == math.inf
