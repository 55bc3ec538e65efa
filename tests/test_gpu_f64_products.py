"""Double products (nmf_dense_AF, nmf_dense_AtF) around the tiles and the
launch shapes of the kernels (16, 32 and 64 rows or columns per wave, ragged
last waves, one and two columns, odd row pitches, A past the last-level
cache) against a float64 product of the same matrices."""
import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import U64, step

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 50, 3), (50, 1, 16), (2, 3, 17), (15, 33, 32), (17, 16, 33), (63, 129, 48),
          (129, 255, 64), (257, 65, 65), (1000, 777, 80), (777, 1001, 96), (2049, 300, 112),
          (515, 2051, 128), (3001, 1700, 40), (4099, 8193, 20), (20000, 1703, 50), (8191, 6007, 10)]


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_product(m, n, k, trans):
    step("f64 product %dx%d k=%d trans=%s" % (m, n, k, trans))
    g = torch.Generator(device="cuda").manual_seed(m + 5 * n + 11 * k)
    A = torch.randn(m, n, generator=g, device="cuda", dtype=torch.float64)
    F = torch.randn(m if trans else n, k, generator=g, device="cuda", dtype=torch.float64)
    got = (nmf.nmf_dense_AtF if trans else nmf.nmf_dense_AF)(A, F)
    Ad = A.T if trans else A
    ref, mag = Ad @ F, Ad.abs() @ F.abs()
    K = F.shape[0]
    # both sides carry at most K roundings of the terms' magnitudes
    assert bool(((got - ref).abs() <= 2 * max(K, 8) * U64 * mag).all())
