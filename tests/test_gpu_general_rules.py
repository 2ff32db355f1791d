"""Rules without a kernel of their own -- order 1, the Duffy orders from 7 on,
seven points per triangle -- in both precisions, for blocks whose sub-tiles are
full, ragged and of one column, per block and in a plan, with the transposed
block of the one-pass form; against the oracle.

Plain FP64 within 1e-12 of the block's largest entry: sums of at most 144^2
terms with a few rounding errors each, distances from coordinates of at most 8
triangle sizes.  Mixed within that form's 1e-6 per block plus the FP32
rounding of phases kappa r, r up to 2."""
import numpy as np
import pytest

import oracle
from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu

RULES = [(0, q) for q in (1, 7, 8, 9, 10, 11, 12)] + [(1, 4)]
M = octahedron_sphere(4)
ROWS = np.arange(3, 24, dtype=np.int32)


def _close(got, ref, precision, kappa):
    if precision:
        assert np.linalg.norm(got - ref) <= (1e-6 + 2.0 * kappa * 2.0 ** -24) * np.linalg.norm(ref)
    else:
        assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("rule,q", RULES)
@pytest.mark.parametrize("kernel,kappa", [(0, 0.0), (1, 1.0)])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ncols", [1, 66])
def test_blocks_and_plans(rule, q, kernel, kappa, precision, ncols):
    import torch
    import paper_1510_07244_amd as pk
    cols = np.arange(60, 60 + ncols, dtype=np.int32)
    n = ROWS.size * cols.size
    mesh = pk.Mesh(torch.from_numpy(M.v), torch.from_numpy(M.tri))
    ref = [oracle.block(M.v, M.tri, a, b, kernel=kernel, layer=l, kappa=kappa, rule=rule, q_reg=q, q_sing=2)
           for l in (0, 1) for a, b in ((ROWS, cols), (cols, ROWS))]
    ctx = pk.Context(0)
    ops = [pk.make_op(kernel, l, precision=precision, regular_rule=rule, q_regular=q, q_singular=2, kappa=kappa)
           for l in (0, 1)]
    new = lambda k: torch.full((k,), float("nan"), dtype=pk.out_dtype(ops[0]), device="cuda")
    one, _ = pk.Blocks.from_lists([ROWS], [cols])
    for l in (0, 1):
        out = new(n)
        ctx.assemble_nearfield(mesh, ops[l], one, out)
        ctx.check()
        _close(out.cpu().numpy().reshape(cols.size, -1).T, ref[2 * l], precision, kappa)
        plan_out = new(n)
        plan = pk.Plan(ctx, ops[l], [(mesh, one, plan_out, False)])
        plan.run()
        ctx.check()
        plan.close()
        assert torch.equal(plan_out, out)
    both = pk.Blocks(np.array([0, ROWS.size]), ROWS, np.array([0, ncols]), cols, np.array([0]), np.array([n]))
    outs = new(2 * n), new(2 * n)
    ctx.assemble_nearfield_both(mesh, ops[0], both, *outs)
    ctx.check()
    for l, out in enumerate(outs):
        got = out.cpu().numpy()
        _close(got[:n].reshape(cols.size, -1).T, ref[2 * l], precision, kappa)
        _close(got[n:].reshape(ROWS.size, -1).T, ref[2 * l + 1], precision, kappa)
    ctx.close()


@pytest.mark.parametrize("rule,q", RULES)
@pytest.mark.parametrize("kernel,kappa", [(0, 0.0), (1, 1.0)])
def test_coupling(rule, q, kernel, kappa):
    """Lists without pairs: wider sub-tiles (up to 128 x 96)."""
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(6)
    c = m.v[m.tri].mean(1)
    rows, cols = (np.nonzero(s * c[:, 2] > 0.2)[0][:101].astype(np.int32) for s in (1, -1))
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    blocks, total = pk.Blocks.from_lists([rows], [cols])
    ctx = pk.Context(0)
    for l in (0, 1):
        op = pk.make_op(kernel, l, regular_rule=rule, q_regular=q, q_singular=2, kappa=kappa)
        out = torch.full((total,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
        ctx.assemble_coupling(mesh, op, blocks, out)
        ctx.check()
        ref = oracle.block(m.v, m.tri, rows, cols, kernel=kernel, layer=l, kappa=kappa, rule=rule, q_reg=q,
                           q_sing=2)
        _close(out.cpu().numpy().reshape(cols.size, -1).T, ref, 0, kappa)
    ctx.close()
