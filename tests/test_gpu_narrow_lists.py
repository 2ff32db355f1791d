"""Mirrored lists of few blocks on edges shared by many triangles.  Such a list
counts edge-adjacent pairs twice and is refused where a sub-tile of 64 x 64 lists
more than 4096; lists of few blocks run in narrower sub-tiles, which may be all
edge-adjacent pairs where the full one is not, and must take and refuse the
same blocks.

Entries against the oracle within 1e-12 of the largest (sums of at most 405
terms), also in the mixed form: singular pairs are summed in FP64 there, the
rest stays within its 1e-6."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _fan_and_strays(n, strays):
    """n triangles around one edge, then triangles of their own far away."""
    ang = np.linspace(0.0, 2.0 * np.pi, n, endpoint=False) + 0.1
    v = [[0, 0, 0], [1, 0, 0]] + [[0.5, np.cos(t), np.sin(t)] for t in ang]
    tri = [[0, 1, 2 + k] for k in range(n)]
    for k in range(strays):
        o = np.array([8.0 + 1.5 * (k % 8), 1.5 * (k // 8), 4.0])
        tri.append([len(v), len(v) + 1, len(v) + 2])
        v += [o, o + [1, 0, 0.1], o + [0.2, 1, 0]]
    return np.array(v, dtype=float), np.array(tri, dtype=np.int32)


def _block(pk, v, tri, rows, cols, diag, precision, layer=0, copies=1):
    """The block and its transpose from a mirrored list (copies of it)."""
    import torch
    nr, nc = rows.size, cols.size
    size = nr * nc * (1 if diag else 2)
    rep = lambda a: np.tile(a, copies)
    off = size * np.arange(copies)
    blocks = pk.Blocks(nr * np.arange(copies + 1), rep(rows), nc * np.arange(copies + 1), rep(cols), off,
                       off + (0 if diag else nr * nc))
    op = pk.make_op(pk.LAPLACE, layer, precision=precision, q_regular=3, q_singular=3,
                    near_singular_ratio=0.5 if precision else 0.0)
    mesh = pk.Mesh(torch.from_numpy(v), torch.from_numpy(tri))
    out = torch.full((size * copies,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
    ctx = pk.Context(0)
    try:
        ctx.assemble_nearfield(mesh, op, blocks, out)
        ctx.check()
    finally:
        ctx.close()
    got = out.cpu().numpy().reshape(copies, size)
    assert (got == got[0]).all()
    got = got[0]
    return [got[:nr * nc].reshape(nc, nr).T] + ([] if diag else [got[nr * nc:].reshape(nr, nc).T])


# 2 * 45^2 = 4050 listed pairs of 64 x 64; 2 * 64 * 32 = 4096 of 64 x 32 and of
# 64 x 64 with columns that touch nothing; on the diagonal 2 * 63 * 64 / 2 + 64
@pytest.mark.parametrize("fan_rows,nr,fan_cols,nc", [(45, 64, 45, 64), (64, 64, 32, 32), (64, 64, 32, 64),
                                                     (40, 64, 33, 70)])
@pytest.mark.parametrize("precision", [0, 1])
def test_taken(fan_rows, nr, fan_cols, nc, precision):
    import paper_1510_07244_amd as pk
    f = fan_rows + fan_cols
    v, tri = _fan_and_strays(f, nr + nc - f)
    stray = np.arange(f, len(tri))
    rows = np.concatenate([np.arange(fan_rows), stray[:nr - fan_rows]]).astype(np.int32)
    cols = np.concatenate([np.arange(fan_rows, f), stray[nr - fan_rows:]]).astype(np.int32)
    got = _block(pk, v, tri, rows, cols, False, precision)
    for g, (a, b) in zip(got, ((rows, cols), (cols, rows))):
        ref = oracle.block(v, tri, a, b, q_reg=3, q_sing=3).real
        assert np.abs(g - ref).max() <= (1e-6 if precision else 1e-12) * np.abs(ref).max()


def test_taken_on_the_diagonal():
    import paper_1510_07244_amd as pk
    v, tri = _fan_and_strays(64, 0)
    idx = np.arange(64, dtype=np.int32)
    ref = oracle.block(v, tri, idx, idx, q_reg=3, q_sing=3).real
    got, = _block(pk, v, tri, idx, idx, True, 0)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("copies", [1, 319, 320, 768])
def test_refused_whatever_the_list(copies):
    """2 * 46^2 = 4232 listed pairs, in narrow sub-tiles and in full ones."""
    import paper_1510_07244_amd as pk
    v, tri = _fan_and_strays(92, 36)
    rows = np.r_[0:46, 92:110].astype(np.int32)
    cols = np.r_[46:92, 110:128].astype(np.int32)
    with pytest.raises(pk.BemError) as e:
        _block(pk, v, tri, rows, cols, False, 0, copies=copies)
    assert e.value.code == pk.BEM_EUNSUPPORTED
