"""Small grids (16 lanes per ray, up to 128^2 rays) and the first grid above
them (one lane per ray), on meshes too small for every lane to have a subtree,
with occlusion tests: ids, distances, flags and occlusion bits against the
oracle, by the comparisons and bounds of the full-size traces."""
import numpy as np
import pytest

from paper_2311_13182_amd import scenes as S
from tests._parity import compare_trace, log

pytestmark = pytest.mark.gpu

F_OCCLUDED = 32


@pytest.mark.parametrize("nx,ny,nf", [(1, 1, 3), (2, 3, 12), (5, 1, 17), (33, 31, 1), (33, 31, 2), (40, 3, 31),
                                      (64, 64, 0), (127, 129, 0), (128, 128, 0), (129, 128, 0)])
def test_small_grids(nx, ny, nf):
    import torch
    from oracle import pyoracle as orc
    from paper_2311_13182_amd.sbr import Simulator
    sc = S.room_scene(n_rays=64).with_grid(nx=nx, ny=ny)
    if nf:   # the faces that a coarse trace meets first, so that some rays hit
        first = orc.trace(sc.with_grid(nx=64, ny=64))["tri"]
        ids, n = np.unique(first[first >= 0], return_counts=True)
        f = sc.faces[np.sort(ids[np.argsort(-n, kind="stable")][:nf])]
        sc = S.Scene("small", sc.verts, f.astype(np.int32), sc.radar, sc.chirp, sc.grid)
    sim = Simulator(sc)
    sim.build()
    sim.trace(count=True)
    torch.cuda.synchronize()
    h = sim.hits
    g = {"tri": h.tri.cpu().numpy(), "t": h.t.cpu().numpy().astype(np.float64), "flags": h.flags.cpu().numpy()}
    o = orc.trace(sc)
    n_ok, n_fl = compare_trace(g, o)
    geom = np.logical_or.accumulate(((g["flags"] & 0x1F) != 0) | ((o["flags"] & 0x1F) != 0), axis=0)
    comp = (o["tri"] >= 0) & (g["tri"] == o["tri"]) & ~geom & (o["shadow_edge"] == 0)
    bad = comp & (((g["flags"] & F_OCCLUDED) != 0) != ((o["flags"] & F_OCCLUDED) != 0))
    log(f"trace {nx}x{ny}, {sc.nf} faces: {n_ok} hits checked, {n_fl} flagged, {bad.sum()} occlusion bits differ")
    assert not bad.any()
    assert abs(int(sim.counters[0].item()) - o["queries"]) <= n_fl
    sim.trace()
    assert torch.equal(sim.hits.tri.cpu(), torch.as_tensor(g["tri"]))
