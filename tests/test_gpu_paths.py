"""The path records and the geometry adjoint at the edges of their forms:
antenna counts around the 32 from which the delays and their adjoint sums get
kernels of their own, one TX or one RX, and every bounce count, for conductors
with the vertices' gradient alone and with the radar's as well.

Oracle: FP64 synthesis and central differences on the oracle's own hits.  Cube:
per sample and relative to sum |I^s|, 3.6e-6 of the transform plus
2 pi (S gamma + C) 2^-25 of the records.  Gradient: the bound of the other
difference tests.  The two kernels run the same single-precision geometry in
different order: 1e-4."""
import numpy as np
import pytest

from paper_2311_13182_amd import scenes as S
from tests._parity import device_hits_from_oracle, log, rel_l2

pytestmark = pytest.mark.gpu

GRAD_TOL = 1e-2


@pytest.mark.parametrize("n_tx,n_rx,K", [(1, 1, 1), (1, 20, 2), (20, 1, 3), (2, 15, 5), (2, 16, 6), (3, 11, 7),
                                         (16, 2, 8)])
def test_antennas_and_bounces(n_tx, n_rx, K):
    import torch
    from oracle import pyoracle as orc
    from paper_2311_13182_amd.sbr import Simulator
    sc = S.trihedral_plate().with_grid(nx=33, ny=31, max_bounces=K)
    sc = S.Scene("paths", sc.verts, sc.faces, S.default_radar(n_tx, n_rx), S.Chirp(n_samples=64, n_chirps=4), sc.grid)
    tr = orc.trace(sc)
    p = orc.paths(sc, tr["tri"], tr["flags"])
    ref = orc.synth(sc, p)
    tgt, _, _ = orc.forward(S.jitter(sc, 1e-3, 17))
    sim = Simulator(sc)
    sim.hits = device_hits_from_oracle(tr)
    got = torch.view_as_complex(sim.synth()).cpu().numpy()
    gam = sc.chirp.slope / sc.chirp.fs * 2 * 3.0 / S.C0
    tol = 3.6e-6 + 2 * np.pi * (64 * gam + 4) * 2.0 ** -25
    err = np.abs(got - ref).max() / np.abs(p["amp"]).sum()
    G = torch.as_tensor((2.0 * (ref - tgt)).astype(np.complex64), device="cuda")
    gr = torch.zeros(6, device="cuda")
    lean = sim.backward(G).double().cpu().numpy()
    full = sim.backward(G, grad_radar=gr).double().cpu().numpy()
    fd = orc.fd_grad(sc, tr["tri"], tr["flags"], tgt, h=1e-9).reshape(-1, 3)
    e, d = rel_l2(lean, fd), rel_l2(lean, full)
    log(f"paths {n_tx}x{n_rx} K={K}: cube {err:.2e} ({tol:.2e}), gradient {e:.2e}, lean against full {d:.2e}")
    assert err <= tol and e <= GRAD_TOL and d <= 1e-4
