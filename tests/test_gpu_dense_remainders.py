"""Products of the complex64 operator with 6 and 7 vectors, and with these left
over after 32 and 16, at a size where the vector units take them by default: 11 524
rows fill neither the last workgroup nor the last staged chunk.  Against the
same operator's single-vector product (2e-6, the bound of the other multi-vector
products)."""
import numpy as np
import pytest

from bem_inputs import complex_normal, geodesic_sphere

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    M = P.Mesh.from_inputs(geodesic_sphere(24))
    x = torch.from_numpy(complex_normal((38, 2 * M.n_vertices), seed=8)).cuda()
    one = torch.stack([P.pmchwt_matvec(M, 4.0, 6.0, 1.5, x[r].contiguous(), precision="fp32_dense")
                       for r in range(38)])
    old = P.tune_get("dense.gemm_min_rhs")
    P.tune_set("dense.gemm_min_rhs", 1000)
    yield P, M, x, one.cpu().numpy()
    P.tune_set("dense.gemm_min_rhs", old)


@pytest.mark.parametrize("R", [6, 7, 23, 38])
def test_remainders(setup, R):
    P, M, x, one = setup
    print(R, flush=True)
    P.profile_enable()
    try:
        y = P.pmchwt_matvec(M, 4.0, 6.0, 1.5, x[:R].contiguous(), precision="fp32_dense").cpu().numpy()
        assert P.profile_read("dense_gemv")[1] == 1
    finally:
        P.profile_enable(False)
    err = np.linalg.norm(y - one[:R], axis=1) / np.linalg.norm(one[:R], axis=1)
    assert err.max() <= 2e-6
