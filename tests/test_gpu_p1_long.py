"""Piecewise-linear pair lists of 2^30 pairs and more: a launch has at most 2^32
threads, so such a list must take few lanes per pair.  One point per triangle
and disjoint pairs; 77 GB of local matrices, of which the first, the last and
some in between are compared with a short list's."""
import numpy as np
import pytest

from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


def test_more_than_a_quarter_of_the_threads():
    import torch
    import paper_1510_07244_amd as pk
    n = (1 << 30) + 5
    if torch.cuda.mem_get_info()[0] < 100 * n:
        pytest.skip("less than 107 GB of device memory free")
    m = octahedron_sphere(4)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    op = pk.make_op(pk.LAPLACE, pk.SLP, q_regular=1, q_singular=1)
    ctx = pk.Context(0)
    rows = torch.arange(n, dtype=torch.int32, device="cuda").remainder_(8)
    cols = rows + 64
    some = torch.tensor([0, 1, 5, (1 << 29) + 3, (1 << 30) - 1, n - 2, n - 1], device="cuda")
    short = torch.empty(9 * some.numel(), dtype=torch.float64, device="cuda")
    ctx.p1_pairs(mesh, op, rows[some].contiguous(), cols[some].contiguous(), short)
    out = torch.empty(9 * n, dtype=torch.float64, device="cuda")
    out.view(n, 9)[some] = float("nan")
    ctx.p1_pairs(mesh, op, rows, cols, out)
    ctx.check()
    got, ref = out.view(n, 9)[some].cpu().numpy(), short.view(-1, 9).cpu().numpy()
    del out, rows, cols
    torch.cuda.empty_cache()
    ctx.close()
    assert np.abs(got - ref).max() <= 1e-13 * np.abs(ref).max()
