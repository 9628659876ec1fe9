"""A product of more vectors than a grid has rows (65 535), on the smallest mesh: the
vectors around that number and the last against their single-vector products (2e-6,
the bound of the other multi-vector products)."""
import numpy as np
import pytest

from bem_inputs import complex_normal, icosphere

pytestmark = pytest.mark.gpu


def test_assembled_product_of_65600_vectors():
    import torch
    import paper_2104_04609_amd as P
    mesh = icosphere(0)
    M = P.Mesh.from_inputs(mesh)
    x = torch.from_numpy(complex_normal((65600, 2 * mesh.n_vertices), seed=1)).cuda()
    print(x.shape, flush=True)
    y = P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x, precision="fp32_dense")
    for r in (0, 65534, 65535, 65536, 65599):
        one = P.pmchwt_matvec(M, 2.0, 3.0, 1.5, x[r].contiguous(), precision="fp32_dense")
        a, b = y[r].cpu().numpy(), one.cpu().numpy()
        assert np.linalg.norm(a - b) / np.linalg.norm(b) <= 2e-6
