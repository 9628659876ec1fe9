"""Phases k r far beyond 2^31 steps of the FP64 phase table (k r of 5e7): the
field at distant points and products with a very large wavenumber, against the
oracle.

Field points lie in the plane through the origin across the incident direction,
so that the incident wave is 1 there and leaves the scattered part exactly up to
its own rounding.  Both sides round r to a few parts in 2^53, so the scattered
part may differ by 8 k r 2^-53, and by 4 2^-53 over its size from adding 1.
Products: phases of up to 2 k differ by 8 k 2^-53 times the entries' sums, with
100 for the cancellation in a row."""
import numpy as np
import pytest

from bem_inputs import complex_normal, icosphere

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    return P


@pytest.mark.parametrize("k0", [10.0, -10.0])
@pytest.mark.parametrize("dist", [30.0, 1e6, 1e7, 1e9, 1e12])
def test_field_of_distant_points(P, dist, k0):
    import torch
    from oracle.field import layer_potentials
    mesh = icosphere(2)
    M = P.Mesh.from_inputs(mesh)
    x = 1e4 * complex_normal(2 * mesh.n_vertices, seed=3)
    a = np.array([0.1, 0.9, 2.2, 3.3, 4.7, 5.8])
    pts = dist * np.stack([np.cos(a), np.sin(a), np.zeros(a.size)], 1)
    print(dist, k0, flush=True)
    u, reg = P.pmchwt_field(M, k0, 15.0, 1.5, [0.0, 0.0, 1.0], torch.from_numpy(x).cuda(),
                            torch.from_numpy(pts).cuda())
    assert not reg.any()
    S, D = layer_potentials(mesh, k0, x, pts)
    scattered = D - S
    err = np.linalg.norm(u.cpu().numpy() - 1.0 - scattered) / np.linalg.norm(scattered)
    bound = (8 * abs(k0) * dist + 4 / np.abs(scattered).min()) * 2.0 ** -53 + 1e-12
    print(err, bound)
    assert err <= bound


@pytest.mark.parametrize("R", [1, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp64_dense"])
def test_product_of_a_large_wavenumber(P, prec, R):
    import torch
    from oracle.operators import pmchwt_matrix
    k0, k1, rho = 2e8, 3e8, 1.5
    mesh = icosphere(1)
    N = mesh.n_vertices
    M = P.Mesh.from_inputs(mesh)
    x = complex_normal((R, 2 * N), seed=4)
    print(prec, R, flush=True)
    y = P.pmchwt_matvec(M, k0, k1, rho, torch.from_numpy(x).cuda(), precision=prec).cpu().numpy()
    ref = x @ pmchwt_matrix(mesh, k0, k1, rho).T
    for sl in (slice(0, N), slice(N, 2 * N)):
        err = np.linalg.norm(y[:, sl] - ref[:, sl]) / np.linalg.norm(ref[:, sl])
        print(err)
        assert err <= 100 * 8 * k1 * 2.0 ** -53
