"""Regions of points exactly in a triangle of the surface, where num = 0 and den < 0:
the triangle's angle is 2 pi or -2 pi by the sign of the zero, as atan2 has it, and
the region 1 or 0 with it, in whatever order and ranges the triangles are summed.

Cube [0, 2]^3 in squares of side h = 1 / m, as two triangles each; coordinates are
multiples of a power of two, so that num is exactly zero and has one sign however
its sums are contracted.  Expected: the sum over the triangles of 2 atan2(num, den)
against 2 pi."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    return P


def cube(m):
    """Vertices, outward triangles; m squares along a unit edge."""
    ids, tri = {}, []
    for ax in range(3):
        e, u, v = np.eye(3, dtype=int)[[ax, (ax + 1) % 3, (ax + 2) % 3]]
        for side in (0, 1):
            for i in range(2 * m):
                for j in range(2 * m):
                    o = 2 * m * side * e + i * u + j * v
                    q = [tuple(o), tuple(o + u), tuple(o + u + v), tuple(o + v)]
                    q = [ids.setdefault(p, len(ids)) for p in (q if side else q[::-1])]
                    tri += [(q[0], q[1], q[2]), (q[0], q[2], q[3])]
    return np.array(list(ids), float) / m, np.array(tri, np.int32)


def solid_angle(V, T, p):
    a, b, c = ((V[T[:, i]] - p).T for i in range(3))
    la, lb, lc = (np.sqrt((v * v).sum(0)) for v in (a, b, c))
    num = (a[0] * (b[1] * c[2] - b[2] * c[1]) + a[1] * (b[2] * c[0] - b[0] * c[2]) +
           a[2] * (b[0] * c[1] - b[1] * c[0]))
    den = (la * lb * lc + (a * b).sum(0) * lc + (a * c).sum(0) * lb + (b * c).sum(0) * la)
    return 2.0 * np.arctan2(num, den).sum()


@pytest.mark.parametrize("order", ["as built", "reversed", "shuffled"])
@pytest.mark.parametrize("m", [1, 4])   # 48 triangles (one range) and 768 (12)
def test_regions_of_face_points(P, m, order):
    import torch
    V, T = cube(m)
    if order == "reversed":
        T = T[::-1]
    elif order == "shuffled":
        T = np.random.default_rng(5).permutation(T)
    a, b, c = (V[T[:, i]] for i in range(3))
    pts = np.concatenate([(2 * a + b + c) / 4, (a + 2 * b + c) / 4, (a + b + 2 * c) / 4])
    share = np.array([solid_angle(V, T, p) for p in pts]) / (4 * np.pi)
    assert np.abs(np.abs(share - 0.5) - 0.5).max() < 1e-9
    assert (share > 0.5).any() and (share < 0.5).any()
    print(m, order, len(pts), flush=True)
    M = P.Mesh(V, T)
    x = torch.zeros(2 * len(V), dtype=torch.complex128, device="cuda")
    _, reg = P.pmchwt_field(M, 2.0, 3.0, 1.5, [0.0, 0.0, 1.0], x,
                            torch.from_numpy(np.ascontiguousarray(pts)).cuda())
    assert np.array_equal(reg.cpu().numpy(), (share > 0.5).astype(int))
