"""Entry and piecewise-linear pair lists at the limits between one, 4 and 16
lanes per regular entry, with rules of 1, 7, 9 and 16 points (lanes without a
point), singular pairs among them, in every class of list length.

A list's value of a pair must not depend on the list's length beyond the
rounding of a sum in another order: within 4 nq eps of the entry's own sum of
absolute values, taken as 1e-13 of the largest entry (kernels of one sign;
the double layer's cancel by less than a factor of ten here).  The shortest
list is compared with the oracle at 1e-12."""
import numpy as np
import pytest

import oracle
from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,kappa", [(0, 0.0), (1, 3.0)])
@pytest.mark.parametrize("rule,q", [(0, 1), (0, 3), (0, 4), (1, 4)])
@pytest.mark.parametrize("layer", [0, 1])
def test_lengths(kernel, kappa, rule, q, layer):
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(8)
    rng = np.random.default_rng(3)
    n0 = 301
    rows = rng.integers(0, m.nt, n0).astype(np.int32)
    cols = rng.integers(0, m.nt, n0).astype(np.int32)
    cols[::9] = np.minimum(rows[::9] + rng.integers(0, 3, rows[::9].size), m.nt - 1)
    op = pk.make_op(kernel, layer, regular_rule=rule, q_regular=q, q_singular=3, kappa=kappa)
    ctx = pk.Context(0)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    ref = oracle.entries(m.v, m.tri, rows, cols, kernel=kernel, layer=layer, kappa=kappa, rule=rule,
                         q_reg=q, q_sing=3)
    big = np.abs(ref).max()
    first = first9 = None
    for n in (n0, (1 << 15) - 1, 1 << 15, (1 << 17) - 1, 1 << 17):
        r, c = np.resize(rows, n), np.resize(cols, n)
        out = torch.full((n,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
        tr, tc = torch.from_numpy(r).cuda(), torch.from_numpy(c).cuda()
        ctx.eval_entries(mesh, op, tr, tc, out)
        ctx.check()
        got = out.cpu().numpy()
        if first is None:
            first = got
            assert np.abs(got - ref).max() <= 1e-12 * big
        assert np.abs(got - np.resize(first, n)).max() <= 1e-13 * big, n
        if n <= 1 << 15:  # local matrices: their sums are the entries
            loc = torch.full((9 * n,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
            ctx.p1_pairs(mesh, op, tr, tc, loc)
            ctx.check()
            loc = loc.cpu().numpy().reshape(n, 9)
            assert np.abs(loc.sum(axis=1) - got).max() <= 1e-12 * big
            first9 = loc if first9 is None else first9
            assert np.abs(loc - np.resize(first9, (n, 9))).max() <= 1e-13 * big
    ctx.close()
