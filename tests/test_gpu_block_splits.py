"""Lists of few blocks, whose sub-tiles are dealt to several workgroups,
against the same entries computed in a list long enough for one workgroup per
block: every entry, mirrors included, is computed by the same sums wherever
its sub-tile lies, so plain FP64 Laplace and double complex entries agree to
1e-13 of the largest one (Helmholtz phases may take either form), mixed ones
to that form's 1e-6."""
import numpy as np
import pytest

from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


def _matrix(ctx, pk, mesh, op, size, repeat, nt):
    """The nt x nt matrix from blocks of `size` triangles, the list repeated."""
    import torch
    edges = list(range(0, nt, size)) + [nt]
    idx = [np.arange(a, b, dtype=np.int32) for a, b in zip(edges, edges[1:])]
    pairs = [(r, c) for c in idx for r in idx]
    blocks, total = pk.Blocks.from_lists([r for r, _ in pairs] * repeat, [c for _, c in pairs] * repeat)
    out = torch.full((total,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
    ctx.assemble_nearfield(mesh, op, blocks, out)
    ctx.check()
    flat, got, k = out.cpu().numpy(), np.empty((nt, nt), out.cpu().numpy().dtype), 0
    for r, c in pairs:
        got[np.ix_(r, c)] = flat[k:k + r.size * c.size].reshape(c.size, r.size).T
        k += r.size * c.size
    return got


# 128 triangles: one block, blocks of ragged sizes, blocks below one sub-tile
@pytest.mark.parametrize("size", [128, 100, 65, 31, 7])
@pytest.mark.parametrize("kernel,layer,precision", [(0, 1, 0), (1, 0, 0), (1, 1, 1)])
def test_few_blocks_equal_many(size, kernel, layer, precision):
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(4)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    op = pk.make_op(kernel, layer, precision=precision, q_regular=4, kappa=2.0 * kernel)
    ctx = pk.Context(0)
    want = _matrix(ctx, pk, mesh, op, 16, 8, 128)  # 8 x 64 = 512 blocks
    got = _matrix(ctx, pk, mesh, op, size, 1, 128)
    ctx.close()
    tol = 1e-6 if precision else 1e-13
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


# 320 blocks and more keep their shape, 768 and more one workgroup each
@pytest.mark.parametrize("nblocks", [319, 320, 767, 768, 1023, 1024])
@pytest.mark.parametrize("coupling", [False, True])
def test_lists_around_the_limits(nblocks, coupling):
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(4)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    op = pk.make_op(0, 0, q_regular=3)
    # two kinds of block, alternating: 7 x 90 and 90 x 7, without touching
    # pairs (coupling launches refuse them)
    small = np.arange(7, dtype=np.int32)
    apart = ~np.isin(m.tri, m.tri[small]).any(1)
    large = np.nonzero(apart)[0][:90].astype(np.int32)
    rows = [small if k % 2 else large for k in range(nblocks)]
    cols = [large if k % 2 else small for k in range(nblocks)]
    blocks, total = pk.Blocks.from_lists(rows, cols)
    out = torch.full((total,), float("nan"), dtype=torch.float64, device="cuda")
    ctx = pk.Context(0)
    run = ctx.assemble_coupling if coupling else ctx.assemble_nearfield
    run(mesh, op, blocks, out)
    ctx.check()
    ctx.close()
    got = out.cpu().numpy().reshape(nblocks, 630)
    # the single layer is symmetric: both kinds hold the same entries
    a, b = got[0].reshape(7, 90).T, got[1].reshape(90, 7).T
    scale = np.abs(a).max()
    assert np.abs(a - b.T).max() <= 1e-13 * scale
    assert (got[0::2] == got[0]).all() and (got[1::2] == got[1]).all()


@pytest.mark.parametrize("cols,fits", [(48, True), (56, False)])
def test_requested_shapes_keep_their_limit(cols, fits):
    """Order 5, 64 rows: 79.7 KB at 48 bytes per column point with 48 columns,
    91.7 KB with 56, of 80 KiB."""
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(4)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    op = pk.make_op(0, 0, q_regular=5)
    idx = np.arange(100, dtype=np.int32)
    blocks, total = pk.Blocks.from_lists([idx], [idx])
    out = torch.full((total,), float("nan"), dtype=torch.float64, device="cuda")
    ctx = pk.Context(0)
    make = lambda: pk.Plan(ctx, op, [(mesh, blocks, out, False)], tune=dict(tile_rows=64, tile_cols=cols))
    if fits:
        plan = make()
        plan.run()
        ctx.check()
        plan.close()
        assert torch.isfinite(out).all()
    else:
        with pytest.raises(Exception, match="LDS budget"):
            make()
    ctx.close()
