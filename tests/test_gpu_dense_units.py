"""Products of the complex64 operator with several vectors on the vector units
(every count a launch takes, 2 to 8, and a remainder) and on the matrix units, as
"dense.skinny_min_rhs" asks: vector units below its value, matrix units from it
on, by the count at its default.  Rows that do not fill a workgroup and columns
that do not fill a staged chunk; against the same operator's single-vector product
(2e-6, the bound of the other multi-vector products)."""
import numpy as np
import pytest

from bem_inputs import complex_normal, geodesic_sphere

pytestmark = pytest.mark.gpu

DEFAULT = 24


@pytest.fixture
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    keys = ("dense.skinny_min_rhs", "dense.gemm_min_rhs")
    old = [P.tune_get(k) for k in keys]
    P.tune_set("dense.gemm_min_rhs", 1000)
    yield P
    for k, v in zip(keys, old):
        P.tune_set(k, v)
    P.profile_enable(False)


_MESH = {}


def check(P, n, R):
    """Launches on the vector and on the matrix units of a product of R vectors."""
    import torch
    if n not in _MESH:
        _MESH.clear()
        _MESH[n] = P.Mesh.from_inputs(geodesic_sphere(n))
    M = _MESH[n]
    x = torch.from_numpy(complex_normal((R, 2 * M.n_vertices), seed=R)).cuda()
    one = [P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x[r].contiguous(), precision="fp32_dense")
           for r in range(R)]
    P.profile_enable()
    y = P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x, precision="fp32_dense")
    torch.cuda.synchronize()
    runs = P.profile_read("dense_gemv")[1], P.profile_read("dense_skinny_mfma")[1]
    for r in range(R):
        a, b = y[r].cpu().numpy(), one[r].cpu().numpy()
        assert np.linalg.norm(a - b) / np.linalg.norm(b) <= 2e-6
    return runs


@pytest.mark.parametrize("R", [2, 3, 4, 5, 6, 7, 8, 11, 23])
@pytest.mark.parametrize("n", [2, 5, 10])   # 84, 504 and 2 004 rows
def test_vector_units(P, n, R):
    print(n, R, flush=True)
    P.tune_set("dense.skinny_min_rhs", 1000)
    assert check(P, n, R) == ((R + 7) // 8, 0)


@pytest.mark.parametrize("R", [2, 7, 16, 19])
@pytest.mark.parametrize("n", [2, 10])
def test_matrix_units(P, n, R):
    print(n, R, flush=True)
    P.tune_set("dense.skinny_min_rhs", 2)
    assert check(P, n, R) == (0, (R + 15) // 16)


def test_line_between_the_units(P):
    P.tune_set("dense.skinny_min_rhs", 5)
    assert check(P, 5, 4) == (1, 0)
    assert check(P, 5, 5) == (0, 1)


@pytest.mark.parametrize("R", [3, 16])
def test_default_goes_by_the_count(P, R):
    assert P.tune_get("dense.skinny_min_rhs") == DEFAULT
    assert check(P, 5, R) == ((1, 0) if R == 3 else (0, 1))
