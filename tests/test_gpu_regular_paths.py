"""Variants of the regular sums on the GPU against the oracle: every Duffy
order with a kernel of its own and the general sums (order 1, orders from 7,
seven points per triangle), and for Helmholtz triangles on both sides of the
limit of the short phases (kappa times the distance of a triangle's points
from its centroid at most 3/4) within one block, kappa of either sign, zero
and too small for scaled coordinates.

Plain FP64 within 1e-12 of the block's largest entry (sums of at most 144^2
terms, a few rounding errors each; phases kappa r up to 40 carry kappa r
2^-53); mixed within the form's 1e-6 per block plus the FP32 rounding of
phases kappa r, r up to 2."""
import numpy as np
import pytest

import oracle
from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import paper_1510_07244_amd as pk
    return pk


def _blocks(pk, m, op, rows, cols, both):
    import torch
    ctx = pk.Context(0)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    blocks, total = pk.Blocks.from_lists([rows], [cols])
    outs = [torch.full((total,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
            for _ in range(2 if both else 1)]
    if both:
        ctx.assemble_nearfield_both(mesh, op, blocks, *outs)
    else:
        ctx.assemble_nearfield(mesh, op, blocks, outs[0])
    ctx.check()
    ctx.close()
    return [o.cpu().numpy().reshape(cols.size, rows.size).T for o in outs]


def _check(pk, kappa, rule, q, precision, both, layer=0, kernel=1):
    m = octahedron_sphere(4)
    rows, cols = np.arange(3, 24, dtype=np.int32), np.arange(40, 127, dtype=np.int32)
    op = pk.make_op(kernel, layer, precision=precision, regular_rule=rule, q_regular=q, q_singular=2,
                    kappa=kappa)
    for k, got in enumerate(_blocks(pk, m, op, rows, cols, both)):
        ref = oracle.block(m.v, m.tri, rows, cols, kernel=kernel, layer=k if both else layer,
                           kappa=kappa, rule=rule, q_reg=q, q_sing=2)
        if precision:
            tol = 1e-6 + 2.0 * abs(kappa) * 2.0 ** -24
            assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
        else:
            assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("rule,q", [(0, q) for q in (1, 2, 3, 4, 5, 6, 7, 8, 12)] + [(1, 4)])
@pytest.mark.parametrize("kernel,kappa", [(0, 0.0), (1, 1.0)])
@pytest.mark.parametrize("precision", [0, 1])
def test_every_rule_variant(pk, rule, q, kernel, kappa, precision):
    if precision and q in (7, 8, 12):
        pytest.skip("one of the general sums' orders suffices in FP32")
    for layer in (0, 1):
        _check(pk, kappa, rule, q, precision, False, layer, kernel)
    _check(pk, kappa, rule, q, precision, True, kernel=kernel)


# radii 0.236 .. 0.333: all triangles short up to 2.24, half of them at 2.6
@pytest.mark.parametrize("kappa", [0.0, 1e-13, 1e-9, -1.5, 2.24, -2.24, 2.6, 20.0])
@pytest.mark.parametrize("q", [3, 4])
@pytest.mark.parametrize("precision", [0, 1])
def test_short_and_general_phases(pk, kappa, q, precision):
    for layer in (0, 1):
        _check(pk, kappa, 0, q, precision, False, layer)
    _check(pk, kappa, 0, q, precision, True)


def test_requested_chunk_does_not_change_entries(pk):
    import torch
    m = octahedron_sphere(4)
    op = pk.make_op(pk.LAPLACE, pk.SLP, q_regular=4, q_singular=4)
    ctx = pk.Context(0)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    idx = np.arange(m.nt, dtype=np.int32)
    blocks, total = pk.Blocks.from_lists([idx], [idx])
    ref = torch.zeros(total, dtype=torch.float64, device="cuda")
    ctx.assemble_nearfield(mesh, op, blocks, ref)
    for chunk in (4, 5, 7, 8, 9):
        out = torch.zeros_like(ref)
        plan = pk.Plan(ctx, op, [(mesh, blocks, out, False)], tune=dict(x_chunk=chunk))
        assert plan.config["x_chunk"] == chunk
        plan.run()
        ctx.check()
        assert torch.equal(out, ref), chunk
        plan.close()
    ctx.close()
