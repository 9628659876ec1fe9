"""Regions and fields where the point lists and triangle ranges end: no point
inside any bounding box, all points inside, one point, points of a box but
outside the surface, objects whose triangles alternate (a sum per change of
object), more points than one pass takes.  Regions against the geometry (the
points keep clear of the surfaces), fields against single-point calls (the same
sums in other ranges: 1e-12)."""
import numpy as np
import pytest

from bem_inputs import geodesic_sphere, two_spheres

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    return P


def _field(P, M, k1, rho, pts):
    import torch
    n2 = 2 * M.n_vertices
    rng = np.random.default_rng(7)
    x = torch.from_numpy(rng.normal(size=n2) + 1j * rng.normal(size=n2)).cuda()
    u, r = P.pmchwt_field(M, 2.0 + 0.01j, k1, rho, [0.0, 0.0, 1.0], x,
                          torch.from_numpy(np.ascontiguousarray(pts)).cuda())
    return u.cpu().numpy(), r.cpu().numpy()


@pytest.mark.parametrize("which", ["outside", "inside", "corners", "one", "mixed"])
@pytest.mark.parametrize("n", [1, 4])   # 20 and 320 triangles
def test_sphere_regions(P, n, which):
    mesh = geodesic_sphere(n)
    M = P.Mesh.from_inputs(mesh)
    rng = np.random.default_rng(n)
    d = rng.normal(size=(700, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    inner = d * rng.uniform(0.05, 0.6, 700)[:, None]
    outer = d * rng.uniform(2.0, 4.0, 700)[:, None]
    corner = np.sign(d) * rng.uniform(0.8, 0.84, (700, 3))   # in the box, outside the sphere
    pts, want = {
        "outside": (outer, 0), "inside": (inner, 1), "corners": (corner, 0), "one": (inner[:1], 1),
        "mixed": (np.concatenate([outer[:257], inner[:300], corner[:3]]),
                  np.repeat([0, 1, 0], [257, 300, 3])),
    }[which]
    print(n, which, flush=True)
    u, r = _field(P, M, 3.0 + 0.1j, 1.5, pts)
    assert np.array_equal(r, np.broadcast_to(want, len(pts)))
    for q in (0, len(pts) // 2, len(pts) - 1):
        one, _ = _field(P, M, 3.0 + 0.1j, 1.5, pts[q:q + 1])
        assert abs(one[0] - u[q]) <= 1e-12 * abs(one[0])


def test_objects_with_alternating_triangles(P):
    m = two_spheres(1)
    order = np.argsort(np.concatenate([np.arange(80), np.arange(80) + 0.5]), kind="stable")
    M = P.Mesh(m.vertices, m.triangles[order], m.object_id[order])
    pts = np.array([[0, -1.5, 0.1], [0, 1.5, -0.2], [0.1, 0.2, 0.0], [0, 1.5, 0.6], [3, 3, 3.0]])
    _, r = _field(P, M, [2.5, 2.0], [1.5, 0.8], pts)
    assert r.tolist() == [1, 2, 0, 2, 0]


def test_more_points_than_one_pass(P):
    M = P.Mesh.from_inputs(geodesic_sphere(1))
    rng = np.random.default_rng(0)
    n = (1 << 22) + 3
    d = np.tile(rng.normal(size=(1024, 3)), ((n + 1023) // 1024, 1))[:n]
    d *= np.where(np.arange(n) % 2, 3.0, 0.4)[:, None] / np.linalg.norm(d, axis=1, keepdims=True)
    u, r = _field(P, M, 3.0, 1.5, d)
    assert np.array_equal(r, (np.arange(n) + 1) % 2)
    assert np.abs(u[1 << 22:] - u[:3]).max() <= 1e-12 * np.abs(u[:3]).max()
