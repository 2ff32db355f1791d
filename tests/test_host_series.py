"""Power series of the Helmholtz radial sums: what the terms left out amount
to.  Singular pairs sum

    sum_p ws e^{i p t}   and   sum_p wd (1 - i p t) e^{i p t},   t = kappa |d|,

over a rule's radial nodes by kSeries even and kSeries odd powers of t as long as t^2 stays within the
device code's limit.  Built here from the Gauss nodes of every order and class
in exact arithmetic: what is left out stays below 3e-17 of the sum's modulus and
6e-17 of its real part, as stated beside the code.  No GPU."""
import pathlib
import re
from fractions import Fraction
from math import factorial

import numpy as np
import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_1510_07244_amd" / "csrc"


def _gauss(q):
    x, w = np.polynomial.legendre.leggauss(q)
    return [Fraction(float(v + 1) / 2) for v in x], [Fraction(float(v) / 2) for v in w]


def _nodes(cls, q):
    """(p, ws, wd) of vertex, edge and identical pairs: J |x - y|^-1 and J <x - y,
    n> |x - y|^-3 with the Jacobians xi^3 (eta), xi^3 eta1^2 and xi^3 eta1^2 eta2."""
    x, w = _gauss(q)
    r = range(q)
    if cls == 1:
        return [(x[a], w[a] * x[a] ** 2, w[a] * x[a]) for a in r]
    if cls == 2:
        return [(x[a] * x[b], w[a] * w[b] * x[a] ** 2 * x[b], w[a] * w[b] * x[a]) for a in r for b in r]
    return [(x[a] * x[b] * x[c], w[a] * w[b] * w[c] * x[a] ** 2 * x[b], 0) for a in r for b in r for c in r]


def _limits():
    n = int(re.search(r"kSeries = (\d+);", (CSRC / "bem_internal.h").read_text()).group(1))
    t2 = {float(v) for v in re.findall(r"kappa \* kappa \* pair_extent2\(g\) <= ([\d.]+)",
                                       (CSRC / "bem_device.h").read_text())}
    assert len(t2) == 1
    return n, Fraction(t2.pop())


@pytest.mark.parametrize("cls", [1, 2, 3])
@pytest.mark.parametrize("q", [1, 2, 3, 4, 5, 6, 8])
def test_terms_left_out(cls, q):
    n, t2 = _limits()
    for layer in (0, 1):
        nodes = [(p, w[layer]) for p, *w in _nodes(cls, q)]
        if not any(w for _, w in nodes):
            continue
        # term k of the sum at t: (+-) moment_k t^k / k!, times (1 - k) for the double layer
        term = lambda k: (sum(w * p ** k for p, w in nodes) * (1 - k if layer else 1)
                          * Fraction((-1) ** (k // 2), factorial(k)))
        even = [term(2 * k) * t2 ** k for k in range(2 * n)]
        odd = [term(2 * k + 1) * t2 ** k for k in range(2 * n)]  # without a factor t
        t = float(t2) ** 0.5
        size = np.hypot(float(sum(even)), float(sum(odd)) * t)
        left = np.hypot(float(sum(even[n:])), float(sum(odd[n:])) * t)
        assert left <= 3e-17 * size, layer
        assert abs(float(sum(even[n:]))) <= 6e-17 * abs(float(sum(even))), layer
