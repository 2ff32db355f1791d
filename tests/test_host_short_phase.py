"""The short-phase sine and cosine of the device code (|x| <= 3/4, no
reduction): coefficients in bem_device.h against their construction
(csrc/sincos_minimax.py) and the routine emulated in double precision
against numpy.  No GPU."""
import importlib.util
import pathlib
import re

import numpy as np
import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_1510_07244_amd" / "csrc"


def _coefficients(name, var):
    """Horner coefficients of `var` in the device function, lowest first."""
    text = (CSRC / "bem_device.h").read_text()
    body = text[text.index(f"void {name}("):]
    body = body[:body.index("\n}\n")]
    num = r"(-?0x[0-9a-f.]+p[-+]?\d+|-?\d+\.\d+)f?"
    vals = re.findall(rf"{var} = (?:fmaf?\({var}, r2, )?{num}\)?;", body)
    return [float.fromhex(v) if "0x" in v else float(v) for v in vals][::-1]


@pytest.mark.parametrize("name,typ,deg,bound", [
    ("short_phase", np.float64, (5, 4), (3.3e-18, 4.1e-17)),
    ("short_phase_f32", np.float32, (2, 2), (6.9e-9, 5.0e-10))])
def test_coefficients_are_the_minimax_ones(name, typ, deg, bound):
    spec = importlib.util.spec_from_file_location("sincos_minimax", CSRC / "sincos_minimax.py")
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    for kind, var, d, b in (("sin", "ps", deg[0], bound[0]), ("cos", "pc", deg[1], bound[1])):
        got = _coefficients(name, var)
        if kind == "cos":
            assert got[0] == -0.5
            got = got[1:]
        ref, levelled = gen.coefficients(kind, d, gen.T_SHORT)
        assert got == [float(typ(c)) for c in ref], kind
        assert levelled <= b
        assert gen.max_rel_error(kind, [typ(c) for c in got], T=gen.T_SHORT) <= b, kind


def test_routine_against_numpy():
    # rounding of the final fused multiply-add, half a unit in the last place
    # each, plus the polynomials' errors above
    x = np.linspace(-0.75, 0.75, 200001)
    r2 = x * x
    ps, pc = (np.polynomial.polynomial.polyval(r2, _coefficients("short_phase", v)) for v in ("ps", "pc"))
    assert np.abs(x + x * r2 * ps - np.sin(x)).max() <= 1.2e-16
    assert np.abs(1.0 + r2 * pc - np.cos(x)).max() <= 2.3e-16
