"""Grouped matrix-vector products at the edges of the kernels' pieces: output
and input counts around 8, 16, 64 and 512, empty and repeated blocks, one long
group among short ones (its rows and panels are then taken in turns).

Against numpy within n eps sum |A| |x| per output (n terms, at most 2 blocks
of 512), the rounding bound of a sum in any order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 8, 9, 15, 16, 17, 63, 64, 65, 127, 128, 129, 511, 512]


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("outs", [SIZES, [2] * 40 + [512], [64, 65], [512]])
def test_pieces_against_numpy(cplx, trans, outs):
    import torch
    import paper_1510_07244_amd as pk
    rng = np.random.default_rng(5)
    num = lambda *s: rng.standard_normal(s) + (1j * rng.standard_normal(s) if cplx else 0)
    x, y0 = num(600), num(sum(outs) + 3)
    out_idx = rng.permutation(y0.size)[:sum(outs)]
    grp_ptr, out_ptr, in_ptr, in_idx, a_off, mats = [0], [0], [0], [], [], []
    want, bound, o = y0.copy(), np.zeros(y0.size), 0
    at = 0
    for g, m in enumerate(outs):
        rows = out_idx[out_ptr[-1]:out_ptr[-1] + m]
        for n in (SIZES[(3 * g) % len(SIZES)], 0, SIZES[(5 * g + 4) % len(SIZES)]):
            ids = rng.integers(0, x.size, n)
            A = num(n, m) if trans else num(m, n)
            want[rows] += (A.T if trans else A) @ x[ids]
            bound[rows] += (np.abs(A.T) if trans else np.abs(A)) @ np.abs(x[ids])
            mats.append(A.ravel(order="F"))
            a_off.append(at)
            at += A.size
            in_idx.append(ids)
            in_ptr.append(in_ptr[-1] + n)
        grp_ptr.append(len(a_off))
        out_ptr.append(out_ptr[-1] + m)
    i32 = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.int32).cuda()
    y = torch.from_numpy(y0).cuda()
    ctx = pk.Context(0)
    args = (trans, i32(grp_ptr), i32(out_ptr), i32(out_idx), i32(in_ptr), i32(np.concatenate(in_idx)),
            torch.as_tensor(a_off, dtype=torch.int64).cuda(), torch.from_numpy(np.concatenate(mats)).cuda(),
            torch.from_numpy(x).cuda())
    ctx.gemv_grouped(*args, y)
    ctx.check()
    tol = 4 * 1024 * np.finfo(float).eps * (bound + np.abs(y0))
    assert np.all(np.abs(y.cpu().numpy() - want) <= tol)
    again = torch.from_numpy(y0).cuda()  # fixed order: the same bits
    ctx.gemv_grouped(*args, again)
    assert torch.equal(torch.view_as_real(again) if cplx else again, torch.view_as_real(y) if cplx else y)
    ctx.close()
