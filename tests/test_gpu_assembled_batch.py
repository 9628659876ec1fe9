"""Products of the assembled operators with several vectors: the matrix-core
product at the edges of its tiles (8, 16 and 32 columns of vectors, groups of
32, rows that do not fill a workgroup, a range of K that ends inside a step),
complex64 and complex128, against the same operator's single-vector product.
Bounds: complex128 sums of 2N = 84 to 2 004 products in another order, 1e-13;
complex64 FP32 sums of at most 64 products, 2e-6 (the bound of the other
multi-vector products)."""
import numpy as np
import pytest

from bem_inputs import complex_normal, geodesic_sphere

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    return P


@pytest.mark.parametrize("prec,tol", [("fp32_dense", 2e-6), ("fp64_dense", 1e-13)])
@pytest.mark.parametrize("R", [2, 4, 5, 8, 9, 17, 32, 37])
@pytest.mark.parametrize("n", [2, 5, 10])   # 42, 252 and 1 002 vertices
def test_assembled_batch(P, n, R, prec, tol):
    import torch
    if ("mesh", n) not in _CACHE:
        _CACHE["mesh", n] = P.Mesh.from_inputs(geodesic_sphere(n))
    M = _CACHE["mesh", n]
    n2 = 2 * M.n_vertices
    x = torch.from_numpy(complex_normal((R, n2), seed=R)).cuda()
    print(n, R, prec, flush=True)
    old = P.tune_get("dense.gemm_min_rhs")
    P.tune_set("dense.gemm_min_rhs", 1000)
    try:
        y = P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x, precision=prec).cpu().numpy()
    finally:
        P.tune_set("dense.gemm_min_rhs", old)
    for r in sorted({0, 1, R // 2, R - 1}):
        one = P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x[r].contiguous(), precision=prec).cpu().numpy()
        assert np.linalg.norm(y[r] - one) / np.linalg.norm(one) <= tol


_CACHE = {}
