"""Assembled products of a few vectors with small operators take the form with the
fewest launches: one on the vector units for up to 8 vectors (complex64, 504 rows),
two single products for two (complex128, 324 rows); larger ones do not.  Against the
same operator's single-vector products (2e-6 and 1e-13, the bounds of the other
multi-vector products)."""
import numpy as np
import pytest

from bem_inputs import complex_normal, geodesic_sphere

pytestmark = pytest.mark.gpu

CASES = [   # mesh frequency, operator, vectors, launches on the vector and matrix units
    (5, "fp32_dense", 6, (1, 0)), (5, "fp32_dense", 8, (1, 0)), (5, "fp32_dense", 9, (0, 1)),
    (8, "fp32_dense", 6, (0, 1)), (4, "fp64_dense", 2, (2, 0)), (4, "fp64_dense", 3, (0, 1)),
    (4, "fp64_dense", 18, (2, 1)), (6, "fp64_dense", 2, (0, 1)),
]


@pytest.mark.parametrize("n,prec,R,want", CASES)
def test_launches_and_products(n, prec, R, want):
    import torch
    import paper_2104_04609_amd as P
    M = P.Mesh.from_inputs(geodesic_sphere(n))
    x = torch.from_numpy(complex_normal((R, 2 * M.n_vertices), seed=R)).cuda()
    one = [P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x[r].contiguous(), precision=prec) for r in range(R)]
    print(n, prec, R, flush=True)
    names = {"fp32_dense": ("dense_gemv", "dense_skinny_mfma"),
             "fp64_dense": ("dense_gemv_fp64", "dense_skinny_mfma64")}[prec]
    P.profile_enable()
    try:
        y = P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x, precision=prec)
        torch.cuda.synchronize()
        assert tuple(P.profile_read(k)[1] for k in names) == want
    finally:
        P.profile_enable(False)
    for r in range(R):
        a, b = y[r].cpu().numpy(), one[r].cpu().numpy()
        assert np.linalg.norm(a - b) / np.linalg.norm(b) <= (2e-6 if prec == "fp32_dense" else 1e-13)
