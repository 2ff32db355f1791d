"""Mean error of mixed entries: the FP32 rounding of an entry's sum is of either
sign, so its mean over many entries shrinks with their number, unless the
rule's own weights were rounded to a wrong sum.

Two patches far apart, where the kernel hardly varies and every entry's
relative error is that of its weights, distances and sum.  The mean over 10 000
entries of at least 7^2 point pairs each stays within a quarter of a rounding,
2^-26 = 1.5e-8, which is left to the mean error of the hardware's reciprocal
root; weights rounded one by one are off by 3e-8 (seven points), 3.7e-8 (order
3, products of two) or 1.5e-8 (order 6)."""
import numpy as np
import pytest

import oracle
from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule,q", [(0, q) for q in range(3, 13)] + [(1, 4)])
@pytest.mark.parametrize("kernel", [0, 1])
def test_mean_error(rule, q, kernel):
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(16)
    r = np.linalg.qr(np.random.default_rng(q).standard_normal((3, 3)))[0]
    v = np.ascontiguousarray((m.v * [1.0, 0.9, 1.2]) @ r.T)
    z = m.v[m.tri].mean(1)[:, 2]
    rows, cols = np.argsort(z)[:100].astype(np.int32), np.argsort(-z)[:100].astype(np.int32)
    kappa = 0.3 * kernel
    op = pk.make_op(kernel, pk.SLP, precision=pk.MIXED, regular_rule=rule, q_regular=q, q_singular=2, kappa=kappa)
    blocks, total = pk.Blocks.from_lists([rows], [cols])
    out = torch.full((total,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
    ctx = pk.Context(0)
    ctx.assemble_nearfield(pk.Mesh(torch.from_numpy(v), torch.from_numpy(m.tri)), op, blocks, out)
    ctx.check()
    ctx.close()
    ref = oracle.block(v, m.tri, rows, cols, kernel=kernel, kappa=kappa, rule=rule, q_reg=q, q_sing=2)
    got = out.cpu().numpy().reshape(cols.size, rows.size).T
    assert abs((got / ref - 1.0).real.mean()) <= 2.0 ** -26
