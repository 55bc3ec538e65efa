"""The MU row update's two splits of a factor into blocks (up to 2048, 3072 or
8192 rows by rank, and above), at the edges of their blocks and of the rule
between them, and the Gram shares that small problems' updates add themselves
(up to 64 at the smallest padded rank), in the order of the separate sum."""
import numpy as np
import pytest

import oracle
import paper_1609_09154_amd as nmf
from synth import uniform
from tests.gpu_util import U32, U64, host, rel_diff, step, to_dev

pytestmark = pytest.mark.gpu

DT = {"f32": (np.float32, U32), "f64": (np.float64, U64)}


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("k", [1, 16, 17, 33, 48, 64])
def test_update_mu_blocks(dt, k):
    npdt, u = DT[dt]
    H = uniform((k, 3 * k + 5), seed=k)
    G = (H @ H.T).astype(npdt)
    for rows in (1, 16, 17, 33, 2048, 2049, 3072, 3073, 8192, 8193):
        P = (uniform((rows, 3 * k + 5), seed=rows + k) @ H.T).astype(npdt)
        X = uniform((rows, k), seed=rows + 2 * k).astype(npdt)
        Xd = to_dev(X, npdt)
        step("mu row blocks %s rows=%d k=%d" % (dt, rows, k))
        nmf.nmf_update("mu", to_dev(G, npdt), to_dev(P, npdt), Xd)
        ref = oracle.mu_update_W(X.astype(np.float64), G.astype(np.float64), P.astype(np.float64))
        # x p / (x G): a k-term sum, one product and one division
        assert rel_diff(host(Xd), ref) <= 4 * (k + 4) * u, rows


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("m,n,k", [(2048, 2049, 16), (2049, 2048, 10), (513, 8192, 16),
                                   (512, 511, 32)])
def test_shares_inside_the_update_match_the_separate_sum(dt, m, n, k):
    """With the objective on, the Grams are formed apart: the same factors bit
    for bit, with 16, 17 and 64 shares."""
    npdt, _ = DT[dt]
    Ad = to_dev(uniform((m, n), seed=m + n).astype(npdt), npdt)
    W0 = uniform((m, k), seed=k).astype(npdt)
    H0 = uniform((k, n), seed=k + 1).astype(npdt)
    outs = []
    for obj in (False, True):
        step("mu shares %s %dx%d k=%d objective=%s" % (dt, m, n, k, obj))
        Wd, Hd = to_dev(W0, npdt), to_dev(H0, npdt)
        nmf.nmf_dense(Ad, Wd, Hd, algo="mu", iters=4, objective=obj)
        outs.append((host(Wd), host(Hd)))
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    np.testing.assert_array_equal(outs[0][1], outs[1][1])
