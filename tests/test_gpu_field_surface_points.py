"""Regions of points that lie on vertices and edges of the surface, where the
triangles around the point have no solid angle: the other triangles alone
decide, in whatever order and ranges they are summed.

The body is the cube [0, 2]^3 without [1, 2]^3, in squares of side h = 1 / m cut
into two triangles, so that the points are exact and every edge length is a power
of two.  Expected: the sum over the triangles of 2 atan2(num, den) against 2 pi, a
triangle with num = den = 0 adding nothing.  Points seen under about half of all
directions (on faces) are left out: rounding decides them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    return P


def notched_cube(m):
    """Vertices, outward triangles; m squares along a unit edge."""
    n = 2 * m
    solid = np.zeros((n + 2,) * 3, bool)   # cells, one layer of air around
    solid[1:-1, 1:-1, 1:-1] = True
    solid[1 + m:-1, 1 + m:-1, 1 + m:-1] = False
    ids, tri = {}, []
    for cell in np.argwhere(solid):
        for ax in range(3):
            for side in (0, 1):
                near = cell.copy()
                near[ax] += 2 * side - 1
                if solid[tuple(near)]:
                    continue
                u, v = np.eye(3, dtype=int)[[(ax + 1) % 3, (ax + 2) % 3]]
                o = cell - 1 + side * np.eye(3, dtype=int)[ax]
                q = [tuple(o), tuple(o + u), tuple(o + u + v), tuple(o + v)]
                q = [ids.setdefault(p, len(ids)) for p in (q if side else q[::-1])]
                tri += [(q[0], q[1], q[2]), (q[0], q[2], q[3])]
    return np.array(list(ids), float) / m, np.array(tri, np.int32)


def solid_angle(V, T, p):
    a, b, c = (V[T[:, i]] - p for i in range(3))
    la, lb, lc = (np.sqrt((v * v).sum(1)) for v in (a, b, c))
    num = (a * np.cross(b, c)).sum(1)
    den = (la * lb * lc + (a * b).sum(1) * lc + (a * c).sum(1) * lb + (b * c).sum(1) * la)
    return 2.0 * np.arctan2(num, den).sum()


@pytest.mark.parametrize("order", ["as built", "reversed", "shuffled"])
@pytest.mark.parametrize("m", [1, 4])   # 48 triangles (one range) and 768 (12)
def test_regions_of_surface_points(P, m, order):
    import torch
    V, T = notched_cube(m)
    if order == "reversed":
        T = T[::-1]
    elif order == "shuffled":
        T = np.random.default_rng(5).permutation(T)
    edges = np.unique(np.sort(np.concatenate([T[:, [0, 1]], T[:, [1, 2]]]), axis=1), axis=0)
    mid = 0.5 * (V[edges[:, 0]] + V[edges[:, 1]])
    along = (V[edges[:, 0]] != V[edges[:, 1]]).sum(1) == 1   # no diagonals
    pts = np.concatenate([V, mid[along]])
    share = np.array([solid_angle(V, T, p) for p in pts]) / (4 * np.pi)
    pts, share = pts[abs(share - 0.5) > 0.1], share[abs(share - 0.5) > 0.1]
    assert share.max() > 0.7 and share.min() < 0.3
    print(m, order, len(pts), flush=True)
    M = P.Mesh(V, T)
    x = torch.zeros(2 * len(V), dtype=torch.complex128, device="cuda")
    _, reg = P.pmchwt_field(M, 2.0, 3.0, 1.5, [0.0, 0.0, 1.0], x,
                            torch.from_numpy(np.ascontiguousarray(pts)).cuda())
    assert np.array_equal(reg.cpu().numpy(), (share > 0.5).astype(int))
