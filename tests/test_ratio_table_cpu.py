"""The table of polynomials with which the Gaussian selector evaluates all pages of a head (csrc/trunc_ratio_coeffs.inc), on the
CPU: evaluated as the kernel does (float32 Horner on s = (1 / (x + K) - mid) / half, products of v) it must reproduce the
truncated Gaussian moments h_n(-x) / phi(x) over the whole range, by numerical quadrature; the reflection the kernel uses for
t > 0 must hold; the moments that the kernel makes of them, in float32 as it does, must be as close as it states on both sides of
zero; and the generator must reproduce the committed file byte for byte."""
import importlib.util
import math
import os
import re

import numpy as np
from scipy import integrate
from scipy.special import ndtr

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_21649_amd", "csrc")
INC = os.path.join(CSRC, "trunc_ratio_coeffs.inc")
NUM = r"[-+]?\d+\.?\d*(?:e[-+]?\d+)?"


def table():
    text = open(INC).read()
    scal = {k: float(v) for k, v in re.findall(r"(kRatioK|kRatioXHi|kRatioMid|kRatioInvHalf) = (" + NUM + ")f", text)}
    deg = [int(x) for x in re.findall(r"\d+", re.search(r"kRatioDeg\[5\] = \{(.*?)\}", text).group(1))]
    rows = re.findall(r"\{((?:\s*" + NUM + r"f,?)+)\}", text[text.index("kRatioCoef[5]"):])
    return scal, deg, [[float(x) for x in re.findall(NUM, r.replace("f", ""))] for r in rows]


def quadrature(n, x):
    return integrate.quad(lambda y: y ** n * math.exp(-x * y - 0.5 * y * y), 0.0, np.inf, epsabs=0.0, epsrel=1e-13, limit=300)[0]


def kernel_ratio(n, x, scal, deg, coef):
    f = np.float32
    fma = lambda a, b, c: f(np.float64(a) * np.float64(b) + np.float64(c))
    v = f(1.0) / f(f(x) + f(scal["kRatioK"]))
    s = fma(v, f(scal["kRatioInvHalf"]), f(-f(scal["kRatioMid"]) * f(scal["kRatioInvHalf"])))
    acc = f(coef[n][deg[n]])
    for c in coef[n][deg[n] - 1::-1]:
        acc = fma(acc, s, f(c))
    for _ in range(n + 1):
        acc = f(acc * v)
    return float(acc)


def test_polynomials_match_quadrature():
    scal, deg, coef = table()
    xs = np.concatenate([np.linspace(0, 4, 121), np.linspace(4, 13, 91)]).astype(np.float32)
    for n in range(5):
        err = np.array([kernel_ratio(n, float(x), scal, deg, coef) / quadrature(n, float(x)) - 1 for x in xs])
        # 1e-7 of the fit; half a unit each in x + K and v, 1.2e-7 together, which the ratio takes to the power n + 3 or less
        assert np.abs(err).max() <= 1e-7 + (n + 3) * 1.2e-7 and np.sqrt(np.mean(err ** 2)) <= 3.5e-7, (n, np.abs(err).max())
        assert all(c == 0.0 for c in coef[n][deg[n] + 1:])


def test_reflection():
    def h(n, t):
        return integrate.quad(lambda z: (t + z) ** n * math.exp(-0.5 * z * z) / math.sqrt(2 * math.pi), -t, 14.0 - t, epsabs=0.0, epsrel=1e-12, limit=300)[0]
    moments = [lambda t: 1.0, lambda t: t, lambda t: t * t + 1, lambda t: t ** 3 + 3 * t, lambda t: t ** 4 + 6 * t * t + 3]
    for t in (0.1, 0.9, 2.5, 6.0):
        for n in range(5):
            assert abs(moments[n](t) - (-1) ** n * h(n, -t) - h(n, t)) <= 1e-9 * h(n, t)
        for n in range(2, 5):                        # the recurrence backwards, all terms positive
            assert abs((h(n, -t) + t * h(n - 1, -t)) / (n - 1) - h(n - 2, -t)) <= 1e-8 * h(n - 2, -t)
    assert abs(quadrature(0, 3.0) * math.exp(-4.5) / math.sqrt(2 * math.pi) / ndtr(-3.0) - 1) <= 1e-12


def kernel_moments(nb, t, scal, deg, coef):
    """trunc_h_all of csrc/select_gauss.hip on a float32 array (its exponential rounded correctly): h_nb, h_(nb-1), h_(nb-2)."""
    f = np.float32
    fma = lambda a, b, c: (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(f)
    x = np.abs(t)
    v = f(1) / (x + f(scal["kRatioK"]))
    s = fma(v, f(scal["kRatioInvHalf"]), f(-f(scal["kRatioMid"]) * f(scal["kRatioInvHalf"])))

    def horner(n):
        acc = np.full_like(t, coef[n][deg[n]])
        for c in coef[n][deg[n] - 1::-1]:
            acc = fma(acc, s, f(c))
        return acc

    u = t * t
    moment = [np.ones_like(t), t, u + f(1), t * (u + f(3)), fma(u, u + f(6), f(3))]           # E[(t + Z)^n]
    phi = np.exp(f(-0.5) * t * t) * f(0.39894228040143268)
    pv = phi
    for _ in range(nb):
        pv = pv * v
    m1, m0 = pv * horner(nb - 1), pv * v * horner(nb)
    pos, sign = t > 0, f(1 if nb % 2 else -1)
    out = [np.where(pos, fma(sign, m0, moment[nb]), m0), np.where(pos, fma(-sign, m1, moment[nb - 1]), m1)]
    if nb >= 2:
        m2 = fma(x, m1, m0) * f(1 / (nb - 1))
        out.append(np.where(pos, fma(sign, m2, moment[nb - 2]), m2))
    return out


def test_moments_match_quadrature():
    scal, deg, coef = table()
    t = np.concatenate([np.linspace(-8, 0, 161), np.linspace(0.01, 12, 121)]).astype(np.float32)
    ref = np.array([[quadrature(n, -float(x)) * math.exp(-0.5 * float(x) ** 2) / math.sqrt(2 * math.pi) for x in t] for n in range(5)])
    for nb in (1, 2, 3, 4):
        for i, got in enumerate(kernel_moments(nb, t, scal, deg, coef)):
            err = np.abs(got / ref[nb - i] - 1)
            # the ratio's bound above (here of nb, of which h_(nb-2) is made), phi's own roundings and half a unit of the exponent t^2 / 2
            limit = 1e-7 + (nb + 3) * 1.2e-7 + 1.2e-7 + 3e-8 * np.minimum(t, 0).astype(np.float64) ** 2
            assert (err <= limit).all(), (nb, nb - i, (err / limit).max())
            assert err[t > -2.5].max() <= 1.1e-6 and err.max() <= 1.8e-6, (nb, nb - i, err.max())


def test_generator_reproduces_the_committed_table(tmp_path):
    spec = importlib.util.spec_from_file_location("gen_trunc_ratio_coeffs", os.path.join(CSRC, "gen_trunc_ratio_coeffs.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    out = tmp_path / "table.inc"
    gen.main(str(out))
    assert out.read_text() == open(INC).read()
