"""A captured single-vector product of one precision, replayed after eager products of
the other: the work lists of the two symmetric kernels differ and each keeps its
own.  Every buffer is grown by an eager product of either precision first; every
replay is compared bit by bit with the eager result on the same input."""
import pytest

from bem_inputs import complex_normal, geodesic_sphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("captured,other", [("fp32", "fp64"), ("fp64", "fp32")])
@pytest.mark.parametrize("n", [6, 12])   # 720 and 2 880 triangles
def test_replay_after_the_other_precision(n, captured, other):
    import torch
    import paper_2104_04609_amd as P
    M = P.Mesh.from_inputs(geodesic_sphere(n))
    x = torch.from_numpy(complex_normal((4, 2 * M.n_vertices), seed=n)).cuda()

    def product(v, prec):
        return P.pmchwt_matvec(M, 2.0, 3.0, 1.5, v, precision=prec)

    product(x[0].contiguous(), other)
    eager = [product(x[r].contiguous(), captured) for r in range(4)]
    torch.cuda.synchronize()
    inp, graph = x[0].clone(), torch.cuda.CUDAGraph()
    print(n, captured, flush=True)
    with torch.cuda.graph(graph):
        out = product(inp, captured)
    for r in range(4):
        product(x[3 - r].contiguous(), other)
        inp.copy_(x[r])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager[r])


@pytest.mark.parametrize("captured", ["fp32", "fp64"])
def test_replay_after_larger_products(captured):
    """Only the captured form has been used before the capture: what products of the
    other precision and of several vectors need later leaves its buffers in place."""
    import torch
    import paper_2104_04609_amd as P
    M = P.Mesh.from_inputs(geodesic_sphere(12))
    x = torch.from_numpy(complex_normal((33, 2 * M.n_vertices), seed=9)).cuda()

    def product(v, prec):
        return P.pmchwt_matvec(M, 2.0, 3.0, 1.5, v, precision=prec)

    eager = [product(x[r].contiguous(), captured) for r in range(5)]
    torch.cuda.synchronize()
    inp, graph = x[0].clone(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = product(inp, captured)
    other = "fp64" if captured == "fp32" else "fp32"
    for r, (prec, R) in enumerate([(other, 1), ("fp32", 8), ("fp64", 8), ("fp32", 16), ("fp32", 33)]):
        print(captured, prec, R, flush=True)
        product(x[:R].contiguous(), prec)
        inp.copy_(x[r])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager[r])
