"""The batch pair kernel (matrix cores) at the edges of its tiles: 16 test
triangles, 4 trial triangles per step, 32 per staged tile, 8, 16 and 32
vectors per launch, remainders of 1 and 2 vectors; real, lossy and
several-material variants, FP32 and FP64, against the oracle's matrix
(tolerances of the matrix-free product: 1e-5 and 1e-10 per block row)."""
import numpy as np
import pytest

from bem_inputs import complex_normal, geodesic_sphere, two_spheres

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    return P


_CASES = {
    "sphere42": (lambda: geodesic_sphere(2), 2.0, [3.0], [1.5]),          # 80 triangles
    "sphere92": (lambda: geodesic_sphere(3), 2.0, [3.0 + 0.2j], [1.5]),   # 180: ragged tiles
    "lossy162": (lambda: geodesic_sphere(4), 2.0 + 0.1j, [3.0], [0.7]),
    "pair84": (lambda: two_spheres(1), 1.5, [2.5, 2.0 + 0.3j], [1.5, 0.8]),
}
_REF = {}


def _case(P, name):
    if name not in _REF:
        from oracle.operators import pmchwt_matrix_multi
        make, k0, k1, rho = _CASES[name]
        mesh = make()
        _REF[name] = (P.Mesh.from_inputs(mesh), mesh.n_vertices,
                      pmchwt_matrix_multi(mesh, k0, k1, rho), k0, k1, rho)
    return _REF[name]


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-5), ("fp64", 1e-10)])
@pytest.mark.parametrize("R", [2, 3, 8, 9, 16, 17, 19, 32, 35])
@pytest.mark.parametrize("name", list(_CASES))
def test_batch_products(P, name, R, prec, tol):
    import torch
    M, N, B, k0, k1, rho = _case(P, name)
    x = np.stack([complex_normal(2 * N, seed=100 + r) for r in range(R)])
    print(name, R, prec, flush=True)
    y = P.pmchwt_matvec_multi(M, k0, k1, rho, torch.from_numpy(x).cuda(), precision=prec).cpu().numpy()
    ref = x @ B.T
    for sl in (slice(0, N), slice(N, 2 * N)):
        err = np.linalg.norm(y[:, sl] - ref[:, sl], axis=1) / np.linalg.norm(ref[:, sl], axis=1)
        assert err.max() <= tol, (err.argmax(), err.max())
