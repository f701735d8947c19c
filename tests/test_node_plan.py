"""The mathematics the Doppler-node form rests on, in NumPy: the width-8 tap
weights compiled into the adjoint (csrc/nu_weights8.h) are the generator's and
follow their kernel, and interpolating e^{2 pi j t nu} from q Chebyshev nodes
stays within the bound by which the library chooses q."""
import importlib.util
import math
import os

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_13182_amd", "csrc")


def _gen():
    spec = importlib.util.spec_from_file_location("gen_nu_weights", os.path.join(CSRC, "gen_nu_weights.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_width_8_weights():
    g = _gen()
    E, O, err = g.fit8()
    with open(os.path.join(CSRC, "nu_weights8.h")) as f:
        assert f.read() == g.header8(E, O, err)
    u = np.random.default_rng(3).uniform(-0.5, 0.5, 5000)
    E, O = E.astype(np.float32).astype(float), O.astype(np.float32).astype(float)
    for t in range(4):
        e, o = np.polyval(E[t][::-1], u * u), u * np.polyval(O[t][::-1], u * u)
        assert np.max(np.abs(e + o - g.psi8(u + 3.5 - t))) < 2e-7
        assert np.max(np.abs(e - o - g.psi8(u - 3.5 + t))) < 2e-7


@pytest.mark.parametrize("x", [0.01, 0.3, 0.47, 2.0, 7.0, 18.0])
def test_chebyshev_nodes_bound(x):
    def bound(q):
        return 4 * sum((0.5 * x) ** k / math.factorial(k) for k in range(q, q + 64))
    q = next(q for q in range(1, 80) if bound(q) <= 1e-7)
    th = math.pi * (2 * np.arange(q) + 1) / (2 * q)
    tau = np.linspace(-1, 1, 2001) + 1e-9
    # L_j = lp y_j / (tau - x_j), lp = prod 2 (tau - x_j), y_j = (-1)^j sin(theta_j) / (2 q)
    d = tau[:, None] - np.cos(th)[None]
    L = np.prod(2 * d, axis=1)[:, None] * ((-1.0) ** np.arange(q) * np.sin(th) / (2 * q)) / d
    for t in np.linspace(-x, x, 9):
        err = np.abs(L @ np.exp(1j * t * np.cos(th)) - np.exp(1j * t * tau)).max()
        assert err <= 1e-7 + 1e-13 * q
