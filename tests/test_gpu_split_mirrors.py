"""Blocks dealt to several workgroups and narrowed sub-tiles, against the same
blocks in a list long enough (768 near-field, 1024 coupling) for one workgroup
per block and full sub-tiles: mirrored blocks off and on the diagonal, both
layers in one pass, coupling with transposes, per-entry orders.  Every entry is
one and the same sum wherever it is computed: equal bit for bit.  The short
list's entries against the oracle at 1e-12 of the largest one."""
import numpy as np
import pytest

import oracle
from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu
M = octahedron_sphere(5)  # 200 triangles
A, B, C = np.arange(0, 90), np.arange(90, 155), np.arange(155, 200)


class _List:
    """copies of the blocks (rows, columns), mirrored if asked: each block's
    output, then its transpose's; a square block on itself is its own."""

    def __init__(self, pk, pairs, mirror, copies):
        rows, cols = [r for r, _ in pairs] * copies, [c for _, c in pairs] * copies
        ptr = lambda x: np.cumsum([0] + [len(i) for i in x])
        off, moff, at = [], [], 0
        for r, c in pairs:
            own = r is c
            off.append(at)
            moff.append(at if own else at + len(r) * len(c))
            at += len(r) * len(c) * (2 if mirror and not own else 1)
        shift = np.repeat(at * np.arange(copies), len(pairs))
        self.size, self.total, self.off, self.moff = at, at * copies, off, moff
        cat = lambda x: np.concatenate(x).astype(np.int32)
        self.blocks = pk.Blocks(ptr(rows), cat(rows), ptr(cols), cat(cols), np.tile(off, copies) + shift,
                                np.tile(moff, copies) + shift if mirror else None)


def _compare(pk, pairs, mirror, op, run, noutputs, limit):
    """Outputs of the short list; asserts the long one's and 320 blocks' equal."""
    import torch
    mesh = pk.Mesh(torch.from_numpy(M.v), torch.from_numpy(M.tri))
    ctx = pk.Context(0)
    first = None
    for copies in (1, -(-320 // len(pairs)), -(-limit // len(pairs))):
        ls = _List(pk, pairs, mirror, copies)
        outs = [torch.full((ls.total,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
                for _ in range(noutputs)]
        run(ctx, mesh, ls, *outs)
        ctx.check()
        outs = [o.view(copies, ls.size) for o in outs]
        first = first or (ls, [o[0].clone() for o in outs])
        for o, f in zip(outs, first[1]):
            assert torch.equal(o, f.expand_as(o)), copies
    ctx.close()
    ls, outs = first
    return ls, [o.cpu().numpy() for o in outs]


def _check(ls, pairs, mirror, out, **kw):
    for (r, c), o, m in zip(pairs, ls.off, ls.moff):
        for a, b, at in ((r, c, o),) + (((c, r, m),) if mirror else ()):
            ref = oracle.block(M.v, M.tri, a.astype(np.int32), b.astype(np.int32), **kw)
            got = out[at:at + a.size * b.size].reshape(b.size, a.size).T
            assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


NEAR = [(A, A), (A, B), (C, C), (B, C)]
OPS = [(0, 0.0), (1, 1.5), (1, 9.0)]


@pytest.mark.parametrize("kernel,kappa", OPS)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("both", [False, True])
def test_near_field_with_mirrors(kernel, kappa, precision, both):
    import paper_1510_07244_amd as pk
    kw = dict(q_regular=3, q_singular=3, kappa=kappa)
    op = pk.make_op(kernel, 0, precision=precision, near_singular_ratio=0.5 if precision else 0.0, **kw)
    run = ((lambda ctx, mesh, ls, a, b: ctx.assemble_nearfield_both(mesh, op, ls.blocks, a, b)) if both else
           (lambda ctx, mesh, ls, a: ctx.assemble_nearfield(mesh, op, ls.blocks, a)))
    ls, outs = _compare(pk, NEAR, True, op, run, 2 if both else 1, 768)
    if not precision:
        for layer, out in enumerate(outs):
            _check(ls, NEAR, True, out, kernel=kernel, layer=layer, kappa=kappa, q_reg=3, q_sing=3)


@pytest.mark.parametrize("kernel,kappa", OPS)
@pytest.mark.parametrize("precision", [0, 1])
def test_coupling_with_transposes(kernel, kappa, precision):
    import paper_1510_07244_amd as pk
    z = M.v[M.tri].mean(1)[:, 2]
    up, down = np.nonzero(z > 0.3)[0], np.nonzero(z < -0.3)[0]
    pairs = [(up, down), (up[:7], down), (down[:33], up[5:70])]
    kw = dict(q_regular=3, q_singular=3, kappa=kappa)
    op = pk.make_op(kernel, 0, precision=precision, near_singular_ratio=0.5 if precision else 0.0, **kw)
    ls, (out,) = _compare(pk, pairs, True, op,
                          lambda ctx, mesh, ls, a: ctx.assemble_coupling(mesh, op, ls.blocks, a), 1, 1024)
    if not precision:
        _check(ls, pairs, True, out, kernel=kernel, layer=0, kappa=kappa, q_reg=3, q_sing=3)


@pytest.mark.parametrize("kernel,kappa", OPS)
@pytest.mark.parametrize("layer", [0, 1])
def test_orders_per_entry(kernel, kappa, layer):
    import torch
    import paper_1510_07244_amd as pk
    pairs = [(A, A), (A, B), (B, C)]
    op = pk.make_op(kernel, layer, q_regular=6, q_singular=3, kappa=kappa)

    def run(ctx, mesh, ls, out):
        one = np.random.default_rng(1).integers(2, 7, ls.size).astype(np.int8)
        orders = torch.from_numpy(np.tile(one, ls.total // ls.size)).cuda()
        ctx.assemble_nearfield_learned(mesh, op, ls.blocks, orders, out)

    _compare(pk, pairs, False, op, run, 1, 768)
