"""The autotuner on two vectors: launches are shared from three vectors on, so one
vector a launch and shared launches are the same work for two, and what their
times happen to be must not keep three vectors (the same entry) from sharing."""
import pytest

from bem_inputs import icosphere

pytestmark = pytest.mark.gpu


@pytest.fixture
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2104_04609_amd as P
    P.tune_clear()
    yield P
    P.tune_clear()


def test_two_vectors_keep_shared_launches(P):
    M = P.Mesh.from_inputs(icosphere(1))
    for q in range(12):
        P.tune_clear()
        e = P.autotune(M, 2.0, 3.0, 1.5, n_rhs=2, expected_matvecs=1)
        print(q, e, flush=True)
        assert e["multi"] == 2
        assert P.tune_lookup(M.n_triangles, 3)[0]["multi"] == 2
