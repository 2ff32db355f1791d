"""The factored singular rules (directions and radial nodes) on the GPU
against the oracle's plain q^4 sums: every class, both kernels, orders from
one point to the largest, and for Helmholtz wave numbers below, across and
above the limit theta = kappa |d| = 2 between the power series and the sum
over radial nodes.

Tolerance 1e-12 of the largest entry: both sides sum the same products in
FP64 (at most 5 q^4 = 1e5 terms of one sign, a few rounding errors each, and
the series' first dropped term is below 1e-17)."""
import numpy as np
import pytest

import oracle
from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def pk():
    import paper_1510_07244_amd as pk
    return pk


def _pairs(m, count):
    """Up to `count` pairs of each class, identical, edge, vertex."""
    shared = (m.tri[:, None, :, None] == m.tri[None, :, None, :]).sum(axis=(2, 3))
    rows, cols = [], []
    for k in (3, 2, 1):
        i, j = np.nonzero(shared == k)
        step = max(1, i.size // count)
        rows.append(i[::step][:count])
        cols.append(j[::step][:count])
    return np.concatenate(rows).astype(np.int32), np.concatenate(cols).astype(np.int32)


# the octahedron sphere's pairs (n = 2) extend over 1.0 .. 1.74
@pytest.mark.parametrize("q", [1, 2, 3, 4, 5, 7, 12])
@pytest.mark.parametrize("kernel,kappa", [(0, 0.0), (1, 0.0), (1, 0.3), (1, 1.3), (1, 9.0)])
def test_singular_entries_every_class(pk, q, kernel, kappa):
    import torch
    m = octahedron_sphere(2)
    r, c = _pairs(m, 6)
    ctx = pk.Context(0)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    for layer in (0, 1):
        op = pk.make_op(kernel, layer, q_regular=2, q_singular=q, kappa=kappa)
        out = torch.full((r.size,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
        ctx.eval_entries(mesh, op, torch.from_numpy(r).cuda(), torch.from_numpy(c).cuda(), out)
        ctx.check()
        ref = oracle.entries(m.v, m.tri, r, c, kernel=kernel, layer=layer, q_reg=2, q_sing=q,
                             kappa=kappa)
        assert np.abs(out.cpu().numpy() - ref).max() <= TOL * np.abs(ref).max(), (layer, q)
    ctx.close()


@pytest.mark.parametrize("kernel,kappa", [(0, 0.0), (1, 0.3), (1, 1.3), (1, 9.0)])
def test_mirrored_one_pass_vertex_pairs(pk, kernel, kappa):
    # a mirrored block: the double layer of the transposed vertex pairs comes
    # from the directions of (i, j)
    import torch
    m = octahedron_sphere(2)
    rows, cols = np.arange(0, 14, dtype=np.int32), np.arange(14, 32, dtype=np.int32)
    n = rows.size * cols.size
    rp, cp = np.array([0, rows.size]), np.array([0, cols.size])
    blocks = pk.Blocks(rp, rows, cp, cols, np.array([0]), np.array([n]))
    op = pk.make_op(kernel, pk.SLP, q_regular=3, q_singular=4, kappa=kappa)
    ctx = pk.Context(0)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    outs = [torch.full((2 * n,), float("nan"), dtype=pk.out_dtype(op), device="cuda") for _ in range(2)]
    ctx.assemble_nearfield_both(mesh, op, blocks, *outs)
    ctx.check()
    for layer, out in enumerate(outs):
        got = out.cpu().numpy()
        for a, b, part in ((rows, cols, got[:n]), (cols, rows, got[n:])):
            ref = oracle.block(m.v, m.tri, a, b, kernel=kernel, layer=layer, q_reg=3, q_sing=4,
                               kappa=kappa)
            assert np.abs(part.reshape(b.size, a.size).T - ref).max() <= TOL * np.abs(ref).max()
    ctx.close()
