"""Green matrices with Green points a small gap above their row triangles,
whose distances lose most if they are formed by a formula that cancels,
against the oracle.

The triangles lie anywhere in space, with vertices of size up to 4 h: as for
close pairs of triangles 28 eps h in a difference of two points on either side
of the comparison; relative to the gap and times the up to seven powers of a
distance in an entry, 512 eps h / gap of each column's largest entry, next to
1e-13 for the sums."""
import numpy as np
import pytest

import oracle
from test_gpu_close_pairs import N, sheets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gap", [1e-2, 1e-4, 1e-6, 1e-8])
@pytest.mark.parametrize("aspect", [1.0, 1e-3])
@pytest.mark.parametrize("kernel,side", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_points_near_their_rows(gap, aspect, kernel, side):
    import torch
    import paper_1510_07244_amd as pk
    v, tri = sheets(1.0, aspect)
    rows = np.arange(2 * N * N, dtype=np.int32)
    p0, e1, e2 = v[tri[rows, 0]], v[tri[rows, 1]] - v[tri[rows, 0]], v[tri[rows, 2]] - v[tri[rows, 1]]
    nrm = np.cross(e1, e2)
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    x, _ = oracle.gauss01(4)
    k = rows % 16  # above one of the rule's points each, alternating sides
    s, t = x[k // 4], x[k // 4] * x[k % 4]
    z = p0 + s[:, None] * e1 + t[:, None] * e2 + (gap / N * (1 - 2 * (rows % 2)))[:, None] * nrm
    zn, zw = -nrm + 0.3 * e1, np.linspace(0.5, 1.5, rows.size)
    dev = lambda a, ty: torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=ty)
    op = pk.make_op(kernel, pk.SLP, q_regular=4, kappa=2.0 * kernel)
    out = torch.full((rows.size * 2 * rows.size,), float("nan"), dtype=pk.out_dtype(op), device="cuda")
    ctx = pk.Context(0)
    mesh = pk.Mesh(torch.from_numpy(v), torch.from_numpy(tri))
    ctx.green_matrix(mesh, op, side, dev([0, rows.size], torch.int32), dev(rows, torch.int32),
                     dev(z[None], torch.float64), dev(zn[None], torch.float64), dev(zw[None], torch.float64),
                     dev([0.25], torch.float64), dev([0], torch.int64), out, max_rows=rows.size)
    ctx.check()
    ctx.close()
    got = out.cpu().numpy().reshape(2 * rows.size, rows.size).T
    ref = oracle.green_matrix(v, tri, rows, z, zn, zw, 0.25, kernel=kernel, kappa=2.0 * kernel, side=side, q=4)
    tol = 1e-13 + 512 * np.finfo(float).eps / gap
    err = np.abs(got - (ref if kernel else ref.real)).max(0)
    assert (err <= tol * np.abs(ref).max(0)).all()
