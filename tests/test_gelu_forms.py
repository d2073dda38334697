"""The GELU forms of the bf16 kernels, evaluated in single precision on the host from the constants in the sources (no GPU needed).

rowlayer.hip and flow.hip run the same layers, for many and for few blocks: whichever a call takes, its error may not be larger than that
of the table in rowlayer.hip.
"""
import math
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_14959_amd", "csrc")
F = np.float32
_phi = np.vectorize(lambda v: 0.5 * math.erfc(-v / math.sqrt(2.0)))


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def _fma(a, b, c):
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(F)


def _body(name):
    src = _source("poly_dev.h")
    at = src.index(f" {name}(")
    return src[at:src.index("\n}\n", at)]


def _numbers(text):
    return [F(v) for v in re.findall(r"-?\d+\.\d+(?:e-?\d+)?(?=f)", text)]


def _poly4(x):
    """gelu_poly4: xc Q(xc^2) with xc cut off, Phi cut off below."""
    body = _body("gelu_poly4")
    clamp = _numbers(re.search(r"fmed3f\(.*?\)", body).group(0))[1]
    horner = _numbers(re.search(r"fmaf\((-?\d[^,]*), s\[i\], (-?\d[^)]*)\)", body).group(0)) + _numbers(re.search(r"c\[\d+\] = \{(.*?)\}", body, re.S).group(1))
    c0 = _numbers(re.search(r"fmaf\(xc\[i\], q\[i\], [^)]*\)", body).group(0))[0]
    xc = np.clip(x, -clamp, clamp)
    return (x * np.maximum(_fma(xc, _horner(horner, (xc * xc).astype(F)), c0), F(0))).astype(F)


def _fine4(x):
    """gelu_fine4: x Q(t) with t cut off, Phi cut off on both sides."""
    body = _body("gelu_fine4")
    k = _numbers(re.search(r"x\[i\] \* [^,]+, -1\.0f\), 1\.0f\)", body).group(0))[0]
    horner = _numbers(re.search(r"fmaf\((-?\d[^,]*), t\[i\], (-?\d[^)]*)\)", body).group(0)) + _numbers(re.search(r"c\[\d+\] = \{(.*?)\}", body, re.S).group(1))
    assert "fmed3f(fmaf(x[i], q[i], 0.5f), 0.f, 1.f)" in body
    t = np.minimum(_fma(x, (x * k).astype(F), F(-1)), F(1))
    return (x * np.clip(_fma(x, _horner(horner, t), F(0.5)), F(0), F(1))).astype(F)


FORMS = {"gelu_poly4": _poly4, "gelu_fine4": _fine4}


def _horner(coefficients, t):
    q = np.full_like(t, coefficients[0])
    for c in coefficients[1:]:
        q = _fma(q, t, c)
    return q


def _table(x):
    t = _fma(np.clip(x, F(-4.5), F(4.5)), F(64), F(288))
    fl = np.floor(t)
    at = np.arange(577)
    p0 = _phi((at - 288) / 64.0).astype(F)
    d = np.append(_phi((at[:-1] + 1 - 288) / 64.0).astype(F) - p0[:-1], F(0)).astype(F)
    i = fl.astype(int)
    return (x * _fma((t - fl).astype(F), d[i], p0[i])).astype(F)


def _errors(f):
    x = np.linspace(-8, 8, 160001).astype(F)
    n = np.random.default_rng(0).standard_normal(100000).astype(F)
    g, gn = x * _phi(x.astype(np.float64)), n * _phi(n.astype(np.float64))
    e = np.abs(f(x) - g)
    big = np.abs(g) > 0.05
    return e.max(), float(np.sqrt(np.mean((f(n) - gn) ** 2))), (e[big] / np.abs(g[big])).max()


def _form_of(kernel):
    return sorted(set(re.findall(r"\b(gelu_(?:poly4|fine4|tab4))\(", _source(kernel))))


@pytest.mark.parametrize("kernel", ["flow.hip"])
def test_kernels_for_few_blocks_are_as_exact_as_the_table(kernel):
    assert _form_of("rowlayer.hip") == ["gelu_tab4"]
    (form,) = _form_of(kernel)
    for mine, table in zip(_errors(FORMS[form]), _errors(_table)):
        assert mine <= table


def test_stated_bounds():
    for form, bounds in (("gelu_poly4", (6.3e-5, 2.0e-5, 3.2e-4)), ("gelu_fine4", (2.4e-5, 2.8e-6, 6e-5))):
        assert all(e <= b for e, b in zip(_errors(FORMS[form]), bounds)), (form, _errors(FORMS[form]))
    assert all(e <= b for e, b in zip(_errors(_table), (2.75e-5, 3.95e-6, 1.4e-4))), _errors(_table)
