"""The FP64 symmetric pair kernel at the edges of its blocks and chunks: 64 to
256 test triangles per workgroup, triangle counts below one block, ragged last
blocks, chunks of 4 triangles to whole tiles, several rounds (bitwise equal to
one); real, lossy and several-material variants.  Against the kernel that
evaluates every ordered pair (the same sums in another order: relative l2
difference of a few units of 2^-53, bound 1e-13) and the oracle (1e-10)."""
import numpy as np
import pytest

from bem_inputs import complex_normal, geodesic_sphere, two_spheres

pytestmark = pytest.mark.gpu
KEYS = ("farfield.block", "farfield.symmetric", "farfield.sym_round_mib")


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    return P


@pytest.fixture
def tune(P):
    old = {k: P.tune_get(k) for k in KEYS}
    yield P.tune_set
    for k, v in old.items():
        P.tune_set(k, v)


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("block", [64, 128, 256])
@pytest.mark.parametrize("name", ["sphere42", "lossy362", "pair324", "sphere1442"])
def test_symmetric_fp64(P, tune, name, block):
    import torch
    from oracle.operators import pmchwt_matrix_multi
    mesh, k0, k1, rho = {
        "sphere42": (geodesic_sphere(2), 2.0, [3.0], [1.5]),              # 80 triangles
        "lossy362": (geodesic_sphere(6), 3.0 + 0.2j, [4.0 + 0.3j], [0.7]),   # 720
        "pair324": (two_spheres(2), 1.5, [2.5, 2.0 + 0.3j], [1.5, 0.8]),   # 640
        "sphere1442": (geodesic_sphere(12), 4.0, [6.0], [1.5]),           # 2 880
    }[name]
    N = mesh.n_vertices
    M = P.Mesh.from_inputs(mesh)
    x = complex_normal(2 * N, seed=31)
    xd = torch.from_numpy(x).cuda()

    def product():
        return P.pmchwt_matvec_multi(M, k0, k1, rho, xd, precision="fp64")

    tune("farfield.block", block)
    print(name, block, flush=True)
    tune("farfield.symmetric", 1)
    y = product()
    tune("farfield.sym_round_mib", 1)   # several rounds from 2 880 triangles on
    assert torch.equal(y, product())
    tune("farfield.symmetric", 0)
    ref = product().cpu().numpy()
    y = y.cpu().numpy()
    for sl in (slice(0, N), slice(N, 2 * N)):
        assert _rel(y[sl], ref[sl]) <= 1e-13
    if N <= 400:
        ref = pmchwt_matrix_multi(mesh, k0, k1, rho) @ x
        for sl in (slice(0, N), slice(N, 2 * N)):
            assert _rel(y[sl], ref[sl]) <= 1e-10
