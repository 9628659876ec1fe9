"""The bottom-subtree plan of a batch is chosen by its number of workgroups: the
same vectors in batches of 1 to 24 (different plans at 2 562 vertices: subtrees of
512 to 4096 rows, fewer and more than 256 workgroups) against one plan for all
(osrc.split 3).  Each is the same direct solve with its sums in another order:
relative difference of a few hundred units of 2^-53 at condition numbers below 1e4,
bound 1e-11."""
import numpy as np
import pytest

from bem_inputs import complex_normal, icosphere, two_spheres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_p,batch", [(1, 1), (4, 1), (4, 4), (8, 6), (4, 16), (4, 24)])
@pytest.mark.parametrize("name", ["sphere642", "pair1284", "sphere2562"])
def test_osrc_plan_by_workgroups(name, n_p, batch):
    import torch
    import paper_2104_04609_amd as P
    mesh = {"sphere642": lambda: icosphere(3), "pair1284": lambda: two_spheres(3, offset=1.5),
            "sphere2562": lambda: icosphere(4)}[name]()
    x = torch.from_numpy(complex_normal((batch, 2 * mesh.n_vertices), seed=batch)).cuda()
    y = P.osrc_apply(P.Mesh.from_inputs(mesh), n_p, np.pi / 3, 6.0, 6.0 + 1.2j, x)
    old = P.tune_get("osrc.split")
    P.tune_set("osrc.split", 3)
    try:
        ref = P.osrc_apply(P.Mesh.from_inputs(mesh), n_p, np.pi / 3, 6.0, 6.0 + 1.2j, x)
    finally:
        P.tune_set("osrc.split", old)
    for r in range(batch):
        assert torch.linalg.norm(y[r] - ref[r]) <= 1e-11 * torch.linalg.norm(ref[r])
