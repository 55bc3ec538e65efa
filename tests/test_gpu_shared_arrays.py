"""Per-step calls whose arrays share memory: the result is that of the same call
on copies (with the outputs written in the order of the arguments), at ranks
that the kernels read in place and at ranks that are padded, for products of
one slab and of several."""
import ctypes

import pytest
import torch

import paper_1609_09154_amd as nmf
from paper_1609_09154_amd import _lib
from tests.gpu_util import step

pytestmark = pytest.mark.gpu

DT = {"f32": torch.float32, "f64": torch.float64}


def rand(g, *shape, dt):
    return torch.rand(*shape, generator=g, device="cuda", dtype=dt) + 0.1


def product(A, F, trans, out):
    """nmf_dense_AF / _AtF into the memory at `out`'s start."""
    L, c = _lib.lib(), nmf._ctx(None, 0)
    f = L.nmf_dense_AtF if trans else L.nmf_dense_AF
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    c.check(f(c.handle, nmf._dtype_code(A), A.shape[0], A.shape[1], p(A), A.stride(0), F.shape[1],
              p(F), F.stride(0), p(out)))


@pytest.mark.parametrize("dt", sorted(DT))
@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("m,n,k", [(5000, 100, 48), (100, 5000, 50), (700, 700, 64), (900, 900, 20)])
def test_product_over_its_inputs(dt, m, n, k, trans):
    step("product over its inputs %s %dx%d k=%d trans=%s" % (dt, m, n, k, trans))
    g = torch.Generator(device="cuda").manual_seed(m + k)
    A, F = rand(g, m, n, dt=DT[dt]), rand(g, m if trans else n, k, dt=DT[dt])
    rows = n if trans else m
    want = (nmf.nmf_dense_AtF if trans else nmf.nmf_dense_AF)(A, F)
    if rows * k <= A.numel():
        B = A.clone()
        product(B, F, trans, B)
        assert torch.equal(B.view(-1)[:rows * k].view(rows, k), want)
    # one buffer for F and, from the same start, the product
    buf = torch.empty(max(F.numel(), rows * k), device="cuda", dtype=DT[dt])
    buf[:F.numel()] = F.view(-1)
    product(A, buf[:F.numel()].view_as(F), trans, buf)
    assert torch.equal(buf[:rows * k].view(rows, k), want)


@pytest.mark.parametrize("dt", sorted(DT))
@pytest.mark.parametrize("algo", ["mu", "hals", "abpp"])
@pytest.mark.parametrize("k", [16, 20, 48, 64])
def test_update_of_shared_arrays(dt, algo, k):
    step("update of shared arrays %s %s k=%d" % (algo, dt, k))
    g = torch.Generator(device="cuda").manual_seed(k)
    H = rand(g, 3 * k, k, dt=DT[dt])
    G = H.T @ H
    if algo != "abpp":    # P = G: a degenerate NNLS, whose pivots may cycle
        want = G.clone()
        nmf.nmf_update(algo, G.clone(), G.clone(), want)
        X = G.clone()
        nmf.nmf_update(algo, X, X, X)
        assert torch.equal(X, want)
    P = rand(g, 500, 3 * k, dt=DT[dt]) @ H
    want = P.clone()
    nmf.nmf_update(algo, G, P.clone(), want)
    X = P.clone()
    nmf.nmf_update(algo, G, X, X)
    assert torch.equal(X, want)


@pytest.mark.parametrize("dt", sorted(DT))
@pytest.mark.parametrize("k", [16, 20, 64])
def test_normalize_of_one_array(dt, k):
    step("normalize of one array %s k=%d" % (dt, k))
    g = torch.Generator(device="cuda").manual_seed(k)
    W = rand(g, 3000, k, dt=DT[dt])
    Wa, Ha = W.clone(), W.clone()
    S, norms = nmf.nmf_hals_normalize(Wa, Ha)
    X = W.clone()
    S2, norms2 = nmf.nmf_hals_normalize(X, X)
    assert torch.equal(X, Ha)    # Ht is written after W
    assert torch.equal(S, S2) and torch.equal(norms, norms2)
