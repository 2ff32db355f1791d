"""A piecewise-linear block uploads its index lists at the call: under stream
capture it is refused, on the capturing stream or passed one, and works again
afterwards."""
import numpy as np
import pytest

from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("passed", [False, True])
def test_capture_is_refused(passed):
    import torch
    import paper_1510_07244_amd as pk
    from paper_1510_07244_amd.p1 import p1_block
    m = octahedron_sphere(3)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    op = pk.make_op(pk.LAPLACE, pk.SLP)
    ctx = pk.Context(0)
    a, b = np.arange(10), np.arange(20, 33)
    ref = p1_block(ctx, mesh, m.tri, op, a, b)  # tables and geometry are there now
    x = torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        x += 1
        with pytest.raises(RuntimeError):
            p1_block(ctx, mesh, m.tri, op, a, b, torch.cuda.current_stream() if passed else None)
    assert torch.equal(p1_block(ctx, mesh, m.tri, op, a, b), ref)
    ctx.check()
    ctx.close()
