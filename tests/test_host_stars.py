"""Triangles around each vertex (the index lists of piecewise-linear blocks)
against a search per vertex, and the calls that are refused: a vertex id
counted from the end, in the list or in a triangle, names no vertex.  No GPU."""
import numpy as np
import pytest

from bem_inputs import octahedron_sphere


@pytest.fixture(scope="module")
def vertex_stars():
    # not while tests are collected: the library would be loaded ahead of torch,
    # and with it another HIP runtime than torch's
    from paper_1510_07244_amd.p1 import vertex_stars
    return vertex_stars


def _search(tri, vertices):
    hits = [[(t, k) for t, c in enumerate(tri.tolist()) for k in range(3) if c[k] == v] for v in vertices]
    tset = sorted({t for h in hits for t, _ in h})
    return (np.cumsum([0] + [len(h) for h in hits]), [tset.index(t) for h in hits for t, _ in h],
            [k for h in hits for _, k in h], tset)


@pytest.mark.parametrize("n,count", [(1, 6), (3, 1), (3, 0), (4, 40)])
@pytest.mark.parametrize("columns", [3, 4])
def test_stars(vertex_stars, n, count, columns):
    m = octahedron_sphere(n)
    rng = np.random.default_rng(n)
    vertices = rng.permutation(m.v.shape[0])[:count]
    tri = np.concatenate([m.tri, np.full((m.nt, columns - 3), m.tri.max(), m.tri.dtype)], axis=1)
    got = vertex_stars(tri, vertices)
    for a, b in zip(got, _search(m.tri, vertices)):
        assert a.dtype == np.int32 and np.array_equal(a, b)


def test_ids_from_the_end_are_refused(vertex_stars):
    m = octahedron_sphere(3)
    last = int(m.tri.max())
    for bad in ([-1], [3, -2], [-1 - last]):
        with pytest.raises(KeyError):
            vertex_stars(m.tri, np.array(bad))
    with pytest.raises(IndexError):
        vertex_stars(m.tri, np.array([last + 1]))
    tri = m.tri.copy()
    tri[5, 1] = -1
    with pytest.raises(KeyError):
        vertex_stars(tri, np.array([last]))
    # named as well, it is that vertex, and the other entry has no triangles
    a, b = vertex_stars(m.tri, np.array([last])), vertex_stars(m.tri, np.array([last, -1]))
    assert np.array_equal(b[0], np.append(a[0], a[0][-1])) and all(np.array_equal(x, y) for x, y in zip(a[1:], b[1:]))


def test_a_vertex_named_twice_keeps_its_last_place(vertex_stars):
    m = octahedron_sphere(3)
    ptr, t_ids, locs, tset = vertex_stars(m.tri, np.array([5, 5, 2]))
    one = vertex_stars(m.tri, np.array([5, 2]))
    assert ptr.tolist() == [0] + one[0].tolist()
    assert all(np.array_equal(x, y) for x, y in zip((t_ids, locs, tset), one[1:]))
