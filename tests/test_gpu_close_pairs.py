"""Facing triangles of two parallel sheets a small gap apart: disjoint pairs
much closer than their size h, whose distances lose most if they are formed
by a formula that cancels.  Entries and piecewise-linear pair lists of every
length class, and the pairs that the mixed form leaves to FP64 as
near-singular, against the oracle.

The sheets lie anywhere in space, with vertices of size up to 4 h.  A point's
coordinates carry about four roundings of eps 4 h / 2 each, a difference of
two points in three coordinates 28 eps h, on either side of the comparison;
relative to the gap and times the four powers of it in the double layer, 256
eps h / gap, next to 1e-13 of the largest entry for the sums.  The mixed form
stores FP32: 2^-23 more."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
N = 4  # squares per side; h = 1 / N


def sheets(gap, aspect):
    """Two sheets of 2 N^2 triangles, triangle k below triangle 2 N^2 + k."""
    X, Y = np.meshgrid(np.arange(N + 1) / N, np.arange(N + 1) / N * aspect, indexing="ij")
    v = np.stack([X.ravel(), Y.ravel(), 0 * X.ravel()], 1)
    at = lambda i, j: i * (N + 1) + j
    t = np.array([c for i in range(N) for j in range(N)
                  for c in ([at(i, j), at(i + 1, j), at(i, j + 1)],
                            [at(i + 1, j), at(i + 1, j + 1), at(i, j + 1)])])
    tri = np.concatenate([t[:, [0, 2, 1]], t + len(v)]).astype(np.int32)
    v = np.concatenate([v, v + [0, 0, gap / N]])
    q = np.linalg.qr(np.random.default_rng(0).standard_normal((3, 3)))[0]
    return np.ascontiguousarray(v @ q.T + 0.3), tri


CASES = [pytest.param(g, a, k, l, id=f"gap{g:g}-aspect{a:g}-{'helmholtz' if k else 'laplace'}-{'dlp' if l else 'slp'}")
         for g in (1e-2, 1e-4, 1e-6, 1e-8) for a in (1.0, 1e-3) for k in (0, 1) for l in (0, 1)]


def _setup(pk, gap, aspect):
    import torch
    v, tri = sheets(gap, aspect)
    i = np.arange(len(tri) // 2, dtype=np.int32)
    return v, tri, pk.Mesh(torch.from_numpy(v), torch.from_numpy(tri)), i, i + i.size


@pytest.mark.parametrize("gap,aspect,kernel,layer", CASES)
def test_entries_and_p1(gap, aspect, kernel, layer):
    import torch
    import paper_1510_07244_amd as pk
    v, tri, mesh, i, j = _setup(pk, gap, aspect)
    op = pk.make_op(kernel, layer, q_regular=4, q_singular=3, kappa=2.0 * kernel)
    kw = dict(kernel=kernel, layer=layer, q_reg=4, q_sing=3, kappa=2.0 * kernel)
    ref = oracle.entries(v, tri, i, j, **kw)
    ref9 = oracle.p1_pairs(v, tri, i, j, **kw).reshape(-1, 9)
    tol = 1e-13 + 256 * np.finfo(float).eps / gap
    ctx = pk.Context(0)
    for n in (i.size, 1 << 15, 1 << 17):
        r, c = (torch.from_numpy(np.resize(a, n)).cuda() for a in (i, j))
        out = torch.full((n,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
        ctx.eval_entries(mesh, op, r, c, out)
        loc = torch.full((9 * n,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
        ctx.p1_pairs(mesh, op, r, c, loc)
        ctx.check()
        assert np.abs(out.cpu().numpy()[:i.size] - ref).max() <= tol * np.abs(ref).max(), n
        assert np.abs(loc.cpu().numpy().reshape(n, 9)[:i.size] - ref9).max() <= tol * np.abs(ref9).max(), n
    ctx.close()


@pytest.mark.parametrize("gap,aspect,kernel,layer", CASES)
def test_mixed_near_singular(gap, aspect, kernel, layer):
    import torch
    import paper_1510_07244_amd as pk
    v, tri, mesh, i, j = _setup(pk, gap, aspect)
    op = pk.make_op(kernel, layer, precision=pk.MIXED, q_regular=4, q_singular=3, kappa=2.0 * kernel,
                    near_singular_ratio=0.5)
    want = lambda l, a, b: oracle.entries(v, tri, a, b, kernel=kernel, layer=l, q_reg=4, q_sing=3,
                                          kappa=2.0 * kernel)
    tol = 2.0 ** -23 + 256 * np.finfo(float).eps / gap
    ctx = pk.Context(0)

    def facing(out, ref):
        got = out.cpu().numpy().reshape(i.size, i.size).diagonal()
        assert np.abs(got - ref).max() <= tol * np.abs(ref).max()

    n = i.size * i.size
    new = lambda k: torch.full((k,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
    one, total = pk.Blocks.from_lists([i], [j])
    out = new(total)
    ctx.assemble_nearfield(mesh, op, one, out)
    ctx.check()
    facing(out, want(layer, i, j))
    if layer == 0:  # both layers in one pass, the transposed block beside
        ptr = np.array([0, i.size])
        both, outs = pk.Blocks(ptr, i, ptr, j, np.array([0]), np.array([n])), (new(2 * n), new(2 * n))
        ctx.assemble_nearfield_both(mesh, op, both, *outs)
        ctx.check()
        for l, out in enumerate(outs):
            facing(out[:n], want(l, i, j))
            facing(out[n:], want(l, j, i))
    ctx.close()
