"""OSRC factors at the edges of their set-up: the update of a column by runs of
up to eight columns (no run, one run that is a whole block, runs of every
remainder) and the device copies of the factors (last workgroups of the
gather, blocks of every width).

Tolerance 1e-10, as for the other comparisons with the oracle's sparse
solves: double precision, shifted systems with condition numbers below 1e4.
"""
import numpy as np
import pytest

from bem_inputs import complex_normal, icosphere, two_spheres

pytestmark = pytest.mark.gpu

CASES = {
    "12_vertices_one_block": (lambda: icosphere(0), 2.0, 3),
    "42_vertices_one_leaf": (lambda: icosphere(1), 3.0, 1),
    "two_objects_of_42": (lambda: two_spheres(1, offset=1.5), 3.0 + 0.2j, 2),
    "162_vertices": (lambda: icosphere(2), 4.0, 5),
    "2562_vertices_lossy": (lambda: icosphere(4), 8.0 + 0.1j, 4),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_osrc_factors_match_oracle(case):
    import torch
    import paper_2104_04609_amd as P
    from oracle.osrc import OSRC, damped_wavenumber
    make, k, n_p = CASES[case]
    mesh = make()
    N = mesh.n_vertices
    keps = damped_wavenumber(k, 0.1)
    x = complex_normal(2 * N, seed=5)
    ref = OSRC(mesh, k, keps, n_p, np.pi / 3).apply(x)
    M = P.Mesh.from_inputs(mesh)
    # a stream of the caller's own: the factors are complete when the call returns
    s = torch.cuda.Stream()
    xd = torch.from_numpy(x).cuda()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        P.osrc_apply(M, n_p, np.pi / 3, k, keps, xd)
    s.synchronize()
    y = P.osrc_apply(M, n_p, np.pi / 3, k, keps, xd).cpu().numpy()   # another stream
    for sl in (slice(0, N), slice(N, 2 * N)):
        err = np.linalg.norm(y[sl] - ref[sl]) / np.linalg.norm(ref[sl])
        assert err <= 1e-10, (case, err)
