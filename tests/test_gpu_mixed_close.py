"""FP32 sums of the mixed form for close pairs left to FP32 (near-singular ratio
0): facing sheets a fraction of their triangle size apart, against the plain
FP32 evaluation of |X|^2 + |Y|^2 - 2 <X, Y> about the row triangle's first vertex
in fused multiply-adds, emulated here with the rest in FP64.  What cancels
there is the distance, and the kernels' polynomial must not lose more than that
and eight FP32 roundings of the rest: root, weights, products, sums, phase and
the stored result.  Either's loss in one position is a matter of luck (the few
distinct differences of a regular sheet), so the largest errors, relative to
the block's largest entry, are compared in their geometric mean over twelve
orientations."""
import numpy as np
import pytest

import oracle
from test_gpu_close_pairs import sheets

pytestmark = pytest.mark.gpu


def _points(v, tri, s, t):
    p = v[tri]
    e1, e2 = p[:, 1] - p[:, 0], p[:, 2] - p[:, 1]
    n = np.cross(e1, e2)
    g = np.linalg.norm(n, axis=1)
    return p[:, 0], s[None, :, None] * e1[:, None] + t[None, :, None] * e2[:, None], g, n / g[:, None]


def _plain_fp32(v, rows, cols, s, t, w, kappa, layer):
    f = np.float32
    vi, X, gi, _ = _points(v, rows, s, t)
    vj, Y, gj, nj = _points(v, cols, s, t)
    x = f(2 * X)
    D = f(2 * (vj[None] - vi[:, None]))
    y = D[:, :, None] + f(2 * Y)[None]
    fma = lambda a, b, c: f(a.astype(float) * b + c)  # the product is exact in FP64
    sq3 = lambda a: fma(a[..., 0], a[..., 0], fma(a[..., 1], a[..., 1], a[..., 2] * a[..., 2]))
    sq = sq3(x)[:, None, :, None] + sq3(y)[:, :, None, :]
    for k in range(3):
        sq = fma(-2 * x[:, None, :, None, k], y[:, :, None, :, k], sq)
    r = np.sqrt(sq.astype(float)) / 2
    k = np.exp(1j * kappa * r) / r
    if layer:
        dn = np.einsum("ijak,jk->ija", (vi[:, None] - vj[None])[:, :, None] + X[:, None], nj)
        k = k * (1 - 1j * kappa * r) / r ** 2 * dn[..., None]
    return np.einsum("a,ijab,b->ij", w, k, w) * gi[:, None] * gj / (4 * np.pi)


@pytest.mark.parametrize("gap", [1.0, 0.3, 0.1, 0.03])
@pytest.mark.parametrize("rule,q", [(0, 2), (0, 3), (0, 4), (0, 5), (0, 6), (0, 8), (1, 4)])
@pytest.mark.parametrize("kernel,layer", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_no_coarser_than_plain(gap, rule, q, kernel, layer):
    import torch
    import paper_1510_07244_amd as pk
    v0, tri = sheets(gap, 1.0)
    h = len(tri) // 2
    rows, cols = np.arange(h, dtype=np.int32), np.arange(h, 2 * h, dtype=np.int32)
    kappa = 2.0 * kernel
    if rule:
        b, w = oracle.tri7()  # barycentric coordinates of (v0, v1, v2)
        s, t, w = b[:, 1] + b[:, 2], b[:, 2], 0.5 * w
    else:
        x, g = oracle.gauss01(q)
        s, t = np.repeat(x, q), np.outer(x, x).ravel()
        w = np.outer(g * x, g).ravel()
    op = pk.make_op(kernel, layer, precision=pk.MIXED, regular_rule=rule, q_regular=q, q_singular=2, kappa=kappa)
    blocks, total = pk.Blocks.from_lists([rows], [cols])
    out = torch.full((total,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
    ctx = pk.Context(0)
    ours, plain = [], []
    for seed in range(12):
        r = np.linalg.qr(np.random.default_rng(seed).standard_normal((3, 3)))[0]
        v = np.ascontiguousarray(v0 @ r.T + 0.1 * seed)
        ctx.assemble_nearfield(pk.Mesh(torch.from_numpy(v), torch.from_numpy(tri)), op, blocks, out)
        ctx.check()
        ref = oracle.block(v, tri, rows, cols, kernel=kernel, layer=layer, kappa=kappa, rule=rule, q_reg=q, q_sing=2)
        big = np.abs(ref).max()
        ours.append(np.abs(out.cpu().numpy().reshape(h, h).T - ref).max() / big)
        plain.append(np.abs(_plain_fp32(v, tri[rows], tri[cols], s, t, w, kappa, layer) - ref).max() / big)
    ctx.close()
    assert np.log(ours).mean() <= np.log(np.array(plain) + 8 * 2.0 ** -24).mean()
