"""Galerkin matrices of piecewise-linear (P1) bases (Sec. 2.2, eq.
reference_integral with low-order polynomial basis functions), driving the
C-ABI: the 3 x 3 local matrices of the triangle pairs (bem_p1_pairs) and
their sums over the triangles around each vertex pair (bem_p1_gather).
This module only builds index lists (the triangles around each vertex) and
orders the calls.
"""
import numpy as np


def vertex_stars(tri, vertices):
    """For the given vertices: the triangles around each (CSR: ptr, triangle
    ids, the vertex's position 0..2 in each), and the sorted set of those
    triangles with the star entries renumbered into it."""
    tri = np.asarray(tri)
    vertices = np.asarray(vertices, dtype=np.int64)
    pos = np.full(int(tri.max()) + 1 if tri.size else 0, -1, dtype=np.int64)
    pos[vertices] = np.arange(vertices.size)
    ends = vertices.size and tri.size and min(vertices.min(), tri.min()) < 0
    if ends:  # ids from the end name no vertex
        named = np.flatnonzero(vertices >= 0)
        pos[vertices[named]] = named
    owner = pos[tri[:, :3]]  # a vertex's number in the list, per corner
    t_ids, locs = np.nonzero(owner >= 0)
    owner = owner[t_ids, locs]
    if ends:
        wrong = vertices[owner] != tri[t_ids, locs]
        if wrong.any():
            raise KeyError(int(tri[t_ids[wrong][0], locs[wrong][0]]))
    order = np.argsort(owner, kind="stable")  # by vertex, then triangle
    used = np.zeros(tri.shape[0], dtype=bool)
    used[t_ids] = True
    tset = np.flatnonzero(used)
    ptr = np.zeros(vertices.size + 1, dtype=np.int32)
    np.cumsum(np.bincount(owner, minlength=vertices.size), out=ptr[1:])
    local = (np.cumsum(used) - 1)[t_ids[order]].astype(np.int32)
    return ptr, local, locs[order].astype(np.int32), tset.astype(np.int32)


def _upload(arrays):
    """int32 device tensors of the arrays: one copy from pinned memory, on the
    current stream and without waiting for it.  Refused under stream capture: the
    pinned memory goes back to its pool, a replay would copy what is there then."""
    import torch
    if torch.cuda.is_current_stream_capturing():
        raise RuntimeError("index lists of a P1 block are uploaded at the call: it cannot be captured")
    sizes = [a.size for a in arrays]
    host = torch.empty(sum(sizes), dtype=torch.int32, pin_memory=True)
    np.concatenate(arrays, out=host.numpy())
    return host.cuda(non_blocking=True).split(sizes)


def p1_block(ctx, mesh, tri, op, row_vertices, col_vertices, stream=None):
    """Dense block (len(row_vertices) x len(col_vertices), a column-major
    device tensor flattened) of the P1 Galerkin matrix of `op`: entry (v, w)
    sums the local matrices of every triangle around v against every
    triangle around w.  mesh: the device Mesh; tri: its host triangles."""
    import torch
    from .h2mv import _on
    rp, rt, rl, rset = vertex_stars(tri, row_vertices)
    cp, ct, cl, cset = vertex_stars(tri, col_vertices)
    nr, nc = rset.size, cset.size
    dt = torch.complex128 if op.kernel == 1 else torch.float64
    with _on(stream):  # copies and allocations in the order of the kernels
        rp, rt, rl, cp, ct, cl, rset, cset = _upload([rp, rt, rl, cp, ct, cl, rset, cset])
        local = torch.empty(9 * nr * nc, dtype=dt, device="cuda")
        ctx.p1_pairs(mesh, op, rset[:, None].expand(nr, nc).reshape(-1),
                     cset.expand(nr, nc).reshape(-1), local, stream)
        out = torch.empty(len(row_vertices) * len(col_vertices), dtype=dt, device="cuda")
        ctx.p1_gather(rp, rt, rl, cp, ct, cl, nr, nc, local, out, stream)
    return out
