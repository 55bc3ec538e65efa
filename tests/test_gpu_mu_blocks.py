"""The MU row update's choice between its two splits of a factor into blocks: by
the rows, the padded rank and the element type, and for float at padded rank 32
by the longer factor too, where the larger blocks' Gram shares are few enough to
be summed inside the update. At each line, whole runs (whose product slabs and
shares follow the same choice) against the oracle's, and against the same run
with the errors on, which forms the Grams apart, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1609_09154_amd as nmf
from synth import init_factors, planted_dense
from tests.gpu_util import U32, U64, host, rel_diff, step, to_dev

pytestmark = pytest.mark.gpu

DT = {"f32": (np.float32, U32), "f64": (np.float64, U64)}


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("m,n,k", [(1024, 1024, 20), (1025, 600, 20), (960, 1088, 30), (3072, 300, 17),
                                   (3073, 300, 32), (16384, 40, 40), (16385, 40, 40),
                                   (8192, 70, 64), (8193, 70, 64), (3073, 300, 60), (2049, 70, 16)])
def test_run_at_the_lines(dt, m, n, k):
    npdt, u = DT[dt]
    iters = 3
    A = planted_dense(m, n, k, seed=m + k).astype(npdt)
    W0, H0 = (x.astype(npdt) for x in init_factors(m, n, k, seed=n + k))
    step("mu run %s %dx%d k=%d" % (dt, m, n, k))
    out = []
    for objective in (False, True):
        W, H = to_dev(W0, npdt), to_dev(H0, npdt)
        nmf.nmf_dense(to_dev(A, npdt), W, H, algo="mu", iters=iters, objective=objective)
        out.append((host(W), host(H)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    W, H, A64 = W0.astype(np.float64), H0.astype(np.float64), A.astype(np.float64)
    for _ in range(iters):
        W = oracle.mu_update_W(W, oracle.gram_fixed_H(H), oracle.product_AHt(A64, H))
        H = oracle.mu_update_H(H, oracle.gram_fixed_W(W), oracle.product_WtA(A64, W))
    # each half-step: a product of n or m terms in slabs, a k-term sum, a quotient;
    # an update passes on at most a few of the roundings it is given
    tol = 8 * (k + 64) * iters * u
    assert rel_diff(out[0][0], W) <= tol and rel_diff(out[0][1], H) <= tol
