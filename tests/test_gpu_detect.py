"""CA-CFAR and the angle stage's conjugate transpose at the edges of their
kernels' tiles, against the oracle.

CFAR: window sums are formed in FP64 from a single-precision power map, so a
cell's ratio is off by that map's rounding: at most Na + 6 roundings of 2^-24
of the cell and of its window's mean.  Every detection must be in the oracle's
list and the other way round except within that distance of the threshold.
Angle stage: each output sums Na products in FP32, relative L2 at most
Na 2^-24 + 2^-22 (the twiddles)."""
import numpy as np
import pytest

from paper_2311_13182_amd import scenes as S

pytestmark = pytest.mark.gpu


def _sim(V, C, Sn, n_angle):
    from paper_2311_13182_amd.sbr import Simulator
    sc = S.single_triangle()
    n_tx = next(t for t in range(1, 21) if V % t == 0 and V // t <= 20)
    sc.radar, sc.chirp = S.default_radar(n_tx, V // n_tx), S.Chirp(n_samples=Sn, n_chirps=C)
    return Simulator(sc, "cuda", n_angle=n_angle, backward=False)


# (Na, C, S, guard, train): tiles of 4 x 64 cells with remainders, windows wider
# than the Doppler axis or the range axis, no guard cells, the widest tiled
# window (16) and one more, one and several block rows of the power map, a
# plane of more than 65,536 cells (several compaction steps per block)
@pytest.mark.parametrize("Na,C,Sn,guard,train", [
    (16, 32, 64, 2, 8), (5, 7, 70, 2, 8), (1, 4, 63, 0, 1), (64, 33, 65, 3, 13), (64, 33, 65, 3, 14), (128, 9, 130, 1, 3),
    (129, 9, 130, 1, 3), (2, 300, 257, 2, 8), (3, 3, 12, 4, 12), (4, 64, 1, 1, 2)])
def test_cfar_tiles(Na, C, Sn, guard, train):
    import torch
    from oracle import pyoracle as orc
    rng = np.random.default_rng(Na * 1000 + C)
    X = (rng.normal(size=(Na, C, Sn)) + 1j * rng.normal(size=(Na, C, Sn))).astype(np.complex64)
    for _ in range(5):
        X[rng.integers(Na), rng.integers(C), rng.integers(Sn)] += 40.0 + 10 * Na ** 0.5
    sim = _sim(Na if Na <= 20 else 1, C, Sn, Na)
    pts, ratio, n = sim.cfar(torch.as_tensor(X, device="cuda"), guard=guard, train=train, pfa=1e-3)
    n = int(n.item())
    pts, ratio = pts[:n].cpu().numpy(), ratio[:n].cpu().numpy()
    o = orc.cfar(X.astype(np.complex128), guard=guard, train=train, pfa=1e-3)
    tol = 2 * (Na + 6) * 2.0 ** -24
    sure = set(zip(*np.nonzero((o["ratio"] > 1 + tol))))
    maybe = set(zip(*np.nonzero((o["ratio"] > 1 - tol))))
    got = [(int(p[1]), int(p[0])) for p in pts]
    assert got == sorted(got) and sure <= set(got) <= maybe
    for p, q in zip(pts, ratio):
        assert int(p[2]) == int(o["argmax"][p[1], p[0]])
        assert abs(q - o["ratio"][p[1], p[0]]) <= tol * o["ratio"][p[1], p[0]]
    # fewer rows than detections: the count is still the total
    few, _, m = sim.cfar(torch.as_tensor(X, device="cuda"), guard=guard, train=train, pfa=1e-3, max_points=2)
    assert int(m.item()) == n and np.array_equal(few[: min(2, n)].cpu().numpy(), pts[:2])


@pytest.mark.parametrize("V,Na,C,Sn", [(1, 1, 3, 5), (1, 7, 8, 16), (12, 64, 8, 40), (16, 16, 4, 16), (17, 37, 4, 33),
                                       (32, 100, 5, 13), (8, 9, 1, 64), (3, 1030, 2, 32)])
def test_angle_adjoint(V, Na, C, Sn):
    import torch
    from oracle import pyoracle as orc
    from paper_2311_13182_amd.sbr import sbr_radar_cube, sbr_radar_cube_2d_bytes
    rng = np.random.default_rng(V)
    X = (rng.normal(size=(Na, C, Sn)) + 1j * rng.normal(size=(Na, C, Sn))).astype(np.complex64)
    ref = orc.radar_cube(X.astype(np.complex128), n_angle=Na, direction=1, V=V)
    out = torch.empty((V, C, Sn, 2), device="cuda")
    scratch = torch.empty(sbr_radar_cube_2d_bytes(V, 1, C, Sn, Na, 1), dtype=torch.uint8, device="cuda")
    sbr_radar_cube(torch.view_as_real(torch.as_tensor(X, device="cuda")).contiguous(), V, C, Sn, Na, 0, 1, out, scratch)
    got = torch.view_as_complex(out).cpu().numpy()
    assert np.linalg.norm(got - ref) <= (Na * 2.0 ** -24 + 2.0 ** -22 + 1e-6) * np.linalg.norm(ref)
