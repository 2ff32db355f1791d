"""Limits of requested sub-tile shapes: a refusal names the request, the limit
lies where 48 bytes (mixed: 32) per column point put it, and rows alone are
taken at every order, with the entries of the default shape."""
import numpy as np
import pytest

from bem_inputs import octahedron_sphere

pytestmark = pytest.mark.gpu


def _run(q, tune, precision=0, both=False, rule=0):
    import torch
    import paper_1510_07244_amd as pk
    m = octahedron_sphere(4)
    mesh = pk.Mesh(torch.from_numpy(m.v), torch.from_numpy(m.tri))
    op = pk.make_op(pk.LAPLACE, pk.SLP, precision=precision, regular_rule=rule, q_regular=q, q_singular=2)
    idx = np.arange(70, dtype=np.int32)
    blocks, total = pk.Blocks.from_lists([idx], [idx + 20])
    out = [torch.full((total,), float("nan"), dtype=pk.out_dtype(op), device="cuda") for _ in range(2)]
    ctx = pk.Context(0)
    entry = (mesh, blocks, out[0], False) + ((pk.BATCH_BOTH, out[1]) if both else ())
    try:
        plan = pk.Plan(ctx, op, [entry], tune=tune)
        plan.run()
        ctx.check()
        plan.close()
    finally:
        ctx.close()
    return out[0]


# columns beside 64 rows within 81920 bytes: order 5 takes 49, 45 with its points
# rounded up to chunks of 7, both layers 48; mixed order 6 takes 46
@pytest.mark.parametrize("q,precision,both,chunk,cols", [(5, 0, False, 0, 49), (5, 0, True, 0, 48),
                                                         (5, 0, False, 7, 45), (6, 1, False, 0, 46)])
def test_limit(q, precision, both, chunk, cols):
    assert bool((_run(q, dict(tile_rows=64, tile_cols=cols, x_chunk=chunk), precision, both)).isfinite().all())
    with pytest.raises(Exception, match="requested tile_cols"):
        _run(q, dict(tile_rows=64, tile_cols=cols + 1, x_chunk=chunk), precision, both)


@pytest.mark.parametrize("rule,q", [(0, q) for q in range(1, 13)] + [(1, 4)])
@pytest.mark.parametrize("precision", [0, 1])
def test_rows_alone(rule, q, precision):
    import torch
    ref = _run(q, {}, precision, rule=rule)
    for rows in (1, 33, 64):
        assert torch.equal(_run(q, dict(tile_rows=rows), precision, rule=rule), ref)
