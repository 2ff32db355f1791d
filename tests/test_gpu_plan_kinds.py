"""Queues of sub-tiles over Helmholtz blocks: the phase kind of a block (short
phases or general ones) is found once per run for all its sub-tiles.  Entries
must equal those of the per-block kernel bit for bit, for blocks of one kind
and of the other in one plan, of one and of many sub-tiles, and again after
the mesh has moved across the limit between the kinds."""
import numpy as np
import pytest

from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


# radii 0.236 .. 0.333: all triangles short up to kappa = 2.24, half of them at 2.6
@pytest.mark.parametrize("kappa", [2.0, 2.6, 20.0, 0.0])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("rows,cols", [(16, 24), (64, 64)])
def test_kinds_follow_the_mesh(kappa, precision, rows, cols):
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(4)
    v = torch.from_numpy(m.v).cuda()
    mesh = pk.Mesh(v, torch.from_numpy(m.tri))
    op = pk.make_op(pk.HELMHOLTZ, pk.SLP, precision=precision, q_regular=3, q_singular=2, kappa=kappa)
    ctx = pk.Context(0)
    all_ = np.arange(m.nt, dtype=np.int32)
    lists = [pk.Blocks.from_lists([all_, all_[:1], all_[5:40]], [all_, all_[7:8], all_[60:]]),
             pk.Blocks.from_lists([all_[k:k + 9] for k in range(0, 117, 9)], [all_[::3]] * 13)]
    ops = [op, pk.make_op(pk.HELMHOLTZ, pk.DLP, precision=precision, q_regular=3, q_singular=2, kappa=kappa)]
    new = lambda n: torch.full((n,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
    outs = [new(total) for _, total in lists]
    plan = pk.Plan(ctx, op, [(mesh, lists[0][0], outs[0], False, pk.BATCH_SLP),
                             (mesh, lists[1][0], outs[1], False, pk.BATCH_DLP)],
                   tune=dict(granularity=2, tile_rows=rows, tile_cols=cols))
    base = mesh.v.clone()
    for scale in (1.0, 0.5, 1.6, 1.0):  # kappa times the radii changes with it
        mesh.v.copy_(base * scale)
        for o in outs:
            o.fill_(float("nan"))
        plan.run()
        ctx.check()
        for o, p, (blocks, total) in zip(outs, ops, lists):
            ref = new(total)
            ctx.assemble_nearfield(mesh, p, blocks, ref)
            ctx.check()
            assert torch.equal(o, ref), scale
    plan.close()
    ctx.close()
