"""The 1D factors of the cell matrix (csrc/op_build.cpp) are their exact values
rounded once.  An entry stands at every cell and in every product of a filter,
so an error of it grows with the degree instead of averaging out.  Built with
g++ and compared with the same factors evaluated here in extended precision."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2203_07820_amd", "csrc", "op_build.cpp")
DRIVER = os.path.join(ROOT, "tests", "native", "tables_1d.cpp")
LD = np.longdouble
U = LD(2) ** -53            # half a unit in the last place of a double, relative
UX = LD(2) ** -64           # the same of the extended format


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    if np.finfo(LD).eps > 2 * UX:
        pytest.skip("no extended precision here")
    out = str(tmp_path_factory.mktemp("t1d") / "tables_1d")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", SRC, DRIVER,
                    "-o", out], check=True)
    return out


def legendre(n, x):
    a, b = np.ones_like(x), x
    for k in range(2, n + 1):
        a, b = b, ((2 * k - 1) * x * b - (k - 1) * a) / LD(k)
    return b, n * (x * b - a) / (x * x - 1)


def factors(p):
    """Stiffness/2 and skew derivative, scaled, with the sums of the absolute
    values of their terms, and the scaled constant function."""
    q = p + 1
    x = np.sort(np.polynomial.legendre.Legendre.basis(p).deriv().roots().real).astype(LD)
    for _ in range(4):      # Newton on P_p', P_p'' from the Legendre equation
        P, d = legendre(p, x)
        x = x - d * (1 - x * x) / (2 * x * d - p * q * P)
    x = np.concatenate([[LD(-1)], (x - x[::-1]) / 2, [LD(1)]])
    P = np.concatenate([[LD((-1) ** p)], legendre(p, x[1:-1])[0], [LD(1)]])
    w = 2 / (LD(p) * q * P * P)
    g = np.polynomial.legendre.leggauss(q)[0].astype(LD)
    for _ in range(4):
        P, d = legendre(q, g)
        g = g - P / d
    gw = 2 / ((1 - g * g) * legendre(q, g)[1] ** 2)
    l, dl, al, adl = (np.zeros((q, q), LD) for _ in range(4))
    for a in range(q):
        o = [b for b in range(q) if b != a]
        den = np.prod([x[a] - x[b] for b in o])
        for i in range(q):
            l[i, a] = np.prod([g[i] - x[b] for b in o]) / den
            t = [np.prod([g[i] - x[b] for b in o if b != c] + [LD(1)]) / den for c in o]
            dl[i, a] = sum(t)
            adl[i, a] = sum(abs(v) for v in t)
    al = abs(l)
    m = np.where((np.arange(q) == 0) | (np.arange(q) == p), w, w / 2)
    s = 1 / np.sqrt(m)[:, None] / np.sqrt(m)
    K, Ka = dl.T @ (gw[:, None] * dl) * s, adl.T @ (gw[:, None] * adl) * s
    G, Ga = l.T @ (gw[:, None] * dl), al.T @ (gw[:, None] * adl)
    return K, Ka, (G - G.T) / 2 * s, (Ga + Ga.T) / 2 * s, np.sqrt(m)


@pytest.mark.parametrize("ncell,L", [(4, 10.0), (7, 7.3)])
@pytest.mark.parametrize("p", range(2, 9))
def test_factors_are_rounded_once(driver, p, ncell, L):
    q = p + 1
    v = np.array([float.fromhex(t) for t in subprocess.check_output([driver, str(p), str(ncell), str(L)],
                                                                   text=True).split()], dtype=LD)
    K, S = v[:q * q].reshape(q, q), v[q * q:2 * q * q].reshape(q, q)
    tK, aK, tS, aS, one = factors(p)
    # one rounding, and what the two evaluations in extended precision may lose:
    # up to 16 q operations on each term
    slack = 2 * 16 * q * UX
    assert (abs(K - tK) <= U * abs(tK) + slack * aK).all()
    assert (abs(S - tS) <= U * abs(tS) + slack * aS).all()
    # the stiffness of a constant is zero up to the same
    assert (abs(K @ one) <= (U * abs(tK) + slack * aK) @ one).all()
