"""Write nu_weights.h: polynomial forms of the 7 kernel-tap weights of the
non-uniform FFT forms as functions of the fractional grid offset.

The kernel is the exponential of semicircle psi(d) = exp(beta (sqrt(1 - (2d/W)^2)
- 1)) for |d| < W/2 (d in grid points), W = 7, beta = 2.3 W.  A point at grid
coordinate x = xr + u (xr = rint(x), u in [-1/2, 1/2]) has taps at
l = xr - 3 + t, t = 0..6, with weights w_t(u) = psi(u + 3 - t).  Since psi is
even, w_{6-t}(u) = w_t(-u); so w_t = E_t(u^2) + u O_t(u^2) and
w_{6-t} = E_t(u^2) - u O_t(u^2) for t = 0, 1, 2, and w_3 = E_3(u^2), each E
of degree 3 and each O of degree 2 in u^2 (degree 6 and 5 in u), fitted by
least squares on a fine grid of u.  The largest error is about 1.4e-6 (about
5e-7 at the edge tap, where psi drops from e^-beta to 0 at the end of its
support).  That is below the kernel's own aliasing error: a type-2 sum
through these weights and through exact psi values differ by under 1e-7 of
sum |h| (S = 64 and 256), while either is about 2e-7 of sum |h| from the
direct sum.

The adjoint over Doppler nodes uses the kernel of width W = 8, beta = 2.3 W
(nu_weights8.h): x = xf + 1/2 + u (xf = floor(x), u in [-1/2, 1/2]), taps at
l = xf - 3 + t, t = 0..7, w_t(u) = psi(u + 7/2 - t) = E_t(u^2) + u O_t(u^2) and
w_{7-t} = E_t(u^2) - u O_t(u^2), t = 0..3, degree 6 and 7 in u (within 9e-8).

Run from the repository root: python paper_2311_13182_amd/csrc/gen_nu_weights.py
"""
from __future__ import annotations

import os

import numpy as np

W = 7
BETA = 2.30 * W
NE, NO = 4, 3   # coefficients of E_t and O_t (powers of u^2)
HERE = os.path.dirname(os.path.abspath(__file__))


def psi(d: np.ndarray) -> np.ndarray:
    x = 2.0 * d / W
    out = np.zeros_like(d, dtype=np.float64)
    m = np.abs(x) < 1.0
    out[m] = np.exp(BETA * (np.sqrt(1.0 - x[m] ** 2) - 1.0))
    return out


def fit():
    u = np.linspace(-0.5, 0.5, 40001)
    u2 = u * u
    E = np.zeros((4, NE))
    O = np.zeros((3, NO))
    err = 0.0
    for t in range(4):
        y = psi(u + 3 - t)
        ye = 0.5 * (y + y[::-1])
        yo = 0.5 * (y - y[::-1])
        E[t] = np.linalg.lstsq(np.vander(u2, NE, increasing=True), ye, rcond=None)[0]
        approx = np.vander(u2, NE, increasing=True) @ E[t]
        if t < 3:
            O[t] = np.linalg.lstsq(u[:, None] * np.vander(u2, NO, increasing=True), yo, rcond=None)[0]
            approx = approx + u * (np.vander(u2, NO, increasing=True) @ O[t])
        err = max(err, float(np.max(np.abs(approx - y))))
    return E, O, err


NE8, NO8 = 4, 4


def psi8(d: np.ndarray) -> np.ndarray:
    x = 2.0 * d / 8
    out = np.zeros_like(d, dtype=np.float64)
    m = np.abs(x) < 1.0
    out[m] = np.exp(2.30 * 8 * (np.sqrt(1.0 - x[m] ** 2) - 1.0))
    return out


def fit8():
    u = np.linspace(-0.5, 0.5, 40001)
    u2 = u * u
    E = np.zeros((4, NE8))
    O = np.zeros((4, NO8))
    err = 0.0
    for t in range(4):
        y = psi8(u + 3.5 - t)
        E[t] = np.linalg.lstsq(np.vander(u2, NE8, increasing=True), 0.5 * (y + y[::-1]), rcond=None)[0]
        O[t] = np.linalg.lstsq(u[:, None] * np.vander(u2, NO8, increasing=True), 0.5 * (y - y[::-1]), rcond=None)[0]
        approx = np.vander(u2, NE8, increasing=True) @ E[t] + u * (np.vander(u2, NO8, increasing=True) @ O[t])
        err = max(err, float(np.max(np.abs(approx - y))))
    return E, O, err


def header8(E: np.ndarray, O: np.ndarray, err: float) -> str:
    def rows(A):
        return ",\n".join("    {" + ", ".join(f"{v:.9e}f" for v in c) + "}" for c in A)
    return "\n".join([
        "// Generated by gen_nu_weights.py (do not edit): least-squares polynomial",
        "// forms of the 8 tap weights of the exponential-of-semicircle kernel of width",
        "// 8, beta = 18.40, in the offset u in [-1/2, 1/2] from the middle between two",
        "// grid points: w_t = E_t(u^2) + u O_t(u^2), w_{7-t} = E_t(u^2) - u O_t(u^2)",
        "// (t < 4); coefficients by ascending power of u^2.  Largest deviation from",
        f"// the kernel on the fitting grid: {err:.2e}.",
        "#pragma once",
        "",
        f"constexpr int kNu8PolyNE = {NE8}, kNu8PolyNO = {NO8};   // coefficients per polynomial",
        f"constexpr float kNu8PolyE[4][{NE8}] = {{",
        rows(E),
        "};",
        f"constexpr float kNu8PolyO[4][{NO8}] = {{",
        rows(O),
        "};",
        "",
    ])


def header(E: np.ndarray, O: np.ndarray, err: float) -> str:
    def row(c):
        return "{" + ", ".join(f"{v:.9e}f" for v in c) + "}"
    lines = [
        "// Generated by gen_nu_weights.py (do not edit): least-squares polynomial",
        "// forms of the 7 tap weights of the non-uniform FFT kernel (exponential of",
        f"// semicircle, W = {W}, beta = {BETA:.2f}) in the fractional grid offset u in",
        "// [-1/2, 1/2]: w_t = E_t(u^2) + u O_t(u^2), w_{6-t} = E_t(u^2) - u O_t(u^2)",
        f"// (t < 3), w_3 = E_3(u^2); coefficients by ascending power of u^2.  Largest",
        f"// deviation from the kernel on the fitting grid: {err:.2e}.",
        "#pragma once",
        "",
        f"constexpr int kNuPolyNE = {NE}, kNuPolyNO = {NO};   // coefficients per polynomial",
        f"constexpr float kNuPolyE[4][{NE}] = {{",
        ",\n".join("    " + row(c) for c in E),
        "};",
        f"constexpr float kNuPolyO[3][{NO}] = {{",
        ",\n".join("    " + row(c) for c in O),
        "};",
        "",
    ]
    return "\n".join(lines)


def main():
    E, O, err = fit()
    text = header(E, O, err)
    path = os.path.join(HERE, "nu_weights.h")
    with open(path, "w") as f:
        f.write(text)
    print(f"wrote {path} (max deviation {err:.2e})")
    E, O, err = fit8()
    path = os.path.join(HERE, "nu_weights8.h")
    with open(path, "w") as f:
        f.write(header8(E, O, err))
    print(f"wrote {path} (max deviation {err:.2e})")


if __name__ == "__main__":
    main()
