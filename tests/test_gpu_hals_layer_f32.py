"""The float HALS layer's results on inputs where an entry of a sweep passes
close to zero. The reverse sweep's mask is x > 0, so there a forward pass whose
products are summed in another order, though as accurate, gives a gradient that
differs by 4e-4 to 1e-2. The recorded results (three ranks: one with a remainder
tile of one column, one of four, one past two whole tiles) are those of products
with the matrix cores' float instruction, slabs and order of K as in
gemm_f32.hip, which the layer keeps: the factors must come out bit for bit, and
the gradients, whose own products no mask follows, within float rounding."""
import os

import numpy as np
import pytest

import paper_1609_09154_amd as nmf
from synth import init_factors, planted_dense, uniform
from tests.conftest import GOLDEN
from tests.gpu_util import host, step, to_dev

pytestmark = pytest.mark.gpu

ITERS, EVERY = 12, 5


@pytest.mark.parametrize("m,n,k,seed", [(150, 113, 17, 1032), (131, 160, 20, 1005),
                                        (200, 96, 33, 1022)])
def test_layer_keeps_its_sums(m, n, k, seed):
    dt = np.float32
    A = to_dev(planted_dense(m, n, k, seed=seed), dt)
    W0, H0 = (to_dev(x, dt) for x in init_factors(m, n, k, seed=seed + 1))
    gW, gH = (to_dev(uniform(s, seed=seed + i) - 0.5, dt) for s, i in (((m, k), 2), ((k, n), 3)))
    step("float hals layer %dx%d k=%d" % (m, n, k))
    W, H, ck = nmf.nmf_hals_unrolled_forward(A, W0, H0, ITERS, ckpt_every=EVERY)
    _, gW0, gH0 = nmf.nmf_hals_unrolled_backward(A, ck, gW, gH, ITERS, ckpt_every=EVERY)
    rec = np.load(os.path.join(GOLDEN, "hals_layer_f32.npz"))
    assert np.array_equal(host(W), rec["W_%d" % seed])
    assert np.array_equal(host(H), rec["H_%d" % seed])
    # 4 T products and sweeps, each adding about k roundings of 2^-24 to what it
    # passes back, in quadrature: 48^(1/2) x 33 x 2^-24 = 1.4e-5
    for x, name in ((gW0, "gW0"), (gH0, "gH0")):
        y = rec["%s_%d" % (name, seed)].astype(np.float64)
        assert np.linalg.norm(host(x) - y) <= 2e-5 * np.linalg.norm(y)
