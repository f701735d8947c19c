"""The work a user of this simulator runs, as cases that can be timed.

Each case is a dict of plain values.  `prepare` makes what a program holds
before the call (scene on the device, Simulator, target signals), `run` is one
pass through the public entry points, `work` counts what the pass cannot do
without and `exact` computes the same outputs in 64 bits with plain torch
(brute-force tracing, direct sums of Eq. 8, autograd through the path
geometry), without the library.

Kinds of pass:
  forward   build the BVH, trace, synthesise the IF cube
  step      forward, IF loss, backward to the vertices (optionally the image too)
  recon     the reconstruction loop's step through torch.autograd (BVH refit,
            trace, synthesis, image, heatmap loss, backward)
  batch     many small requests: build and trace each, one batched synthesis
  geometry  build or refit the BVH and trace
  synth     IF cube of hit records already in hand
  backward  all gradients for hit records and dL/dIF already in hand
  image     radar cube, heatmap loss, conjugate transpose
  detect    radar cube, CFAR, world points
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2311_13182_amd import scenes as S

C0 = 299792458.0
EPS0 = 8.8541878128e-12


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


# ------------------------------------------------------------------ the cases
_BASE = dict(mesh="superquadric", nf=5000, nx=256, ny=256, K=3, n_tx=3, n_rx=4, C=64, S=256, vx=0.0, vz=1.0,
             shadow=False, jitter=False, materials=False, attached=False, planar=False)


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest simulation: corner reflector and plate, one chirp, where
        # launches and host time are what a caller waits for
        _case("trihedral_forward", kind="forward", mesh="trihedral", nf=14, nx=64, ny=64, K=3, n_tx=1, n_rx=4, C=1,
              vz=0.0),
        # one gradient step on a single mid-size object (the icosphere workload)
        _case("icosphere_step", kind="step", mesh="icosphere", nf=20480, nx=512, ny=512, K=3, C=64),
        # one gradient step on the cluttered scene, the headline workload, with
        # the range-Doppler-angle image of the simulated signal
        _case("clutter_step", kind="step", mesh="clutter", nf=51200, nx=2048, ny=2048, K=4, C=128, image=True),
        # one step of the mesh reconstruction loop
        _case("recon_step", kind="recon", mesh="geodesic", nf=9680, nx=1024, ny=1024, K=3, C=64),
        # one step with the 20 x 20 planar imaging array and its 2D angle image
        _case("imaging_step", kind="step", mesh="imaging", nf=20012, nx=512, ny=512, K=2, n_tx=20, n_rx=20, C=16,
              vz=0.5, planar=True, image=True),
        # a burst of small serving requests batched into shared launches
        _case("serving_batch", kind="batch", n=16, nx=256, ny=256, K=2, n_tx=2, C=32, nf=20000),
        # the geometry half of the largest serving request, occlusion-tested
        _case("geometry_200k", kind="geometry", nf=200000, nx=1024, ny=1024, K=4, shadow=True, refit=False),
        # synthesis alone at odd sizes: chirp and sample counts that are no
        # powers of two, a moving lateral scene
        _case("synth_ragged", kind="synth", nf=3000, nx=301, ny=203, K=2, n_tx=2, n_rx=3, C=50, S=200, vx=2.0,
              vz=1.0),
        # every gradient (vertices, materials, pose, velocity, attenuation) of
        # the reparameterised estimator with Fresnel materials
        _case("backward_materials", kind="backward", nf=5000, nx=320, ny=320, K=3, C=32, materials=True,
              attached=True),
        # the image loss and its adjoint at the automotive array's cube size
        _case("image_loss", kind="image", n_tx=3, n_rx=4, C=128, S=256, n_angle=64, window=0),
        # the same with lengths that are no powers of two and a Hann window
        _case("image_ragged", kind="image", n_tx=2, n_rx=4, C=50, S=200, n_angle=48, window=1),
        # detection: image, CFAR, point cloud
        _case("detect", kind="detect", n_tx=3, n_rx=4, C=128, S=256, n_angle=64, window=1),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same kinds with sizes spread over the ranges served: 1k to
    200k triangles, 64^2 to 1448^2 rays, 1 to 4 bounces, 1 to 16 antennas, 1 to
    256 chirps of 16 to 1024 samples, scene speeds up to 15 m/s."""
    kind = rng.choice(["forward", "step", "step", "recon", "batch", "geometry", "synth", "synth", "backward",
                       "backward", "image", "detect"])
    if kind in ("image", "detect"):
        n_tx, n_rx = rng.randint(1, 4), rng.randint(1, 4)
        C, Sn = _logint(rng, 16, 256), _logint(rng, 32, 512)
        if rng.random() < 0.5:
            C, Sn = 1 << round(math.log2(C)), 1 << round(math.log2(Sn))
        return _case(kind=kind, n_tx=n_tx, n_rx=n_rx, C=C, S=Sn, n_angle=rng.choice([16, 32, 37, 48, 64]),
                     window=1 if kind == "detect" else rng.randint(0, 1))
    c = _case(kind=kind, nf=_logint(rng, 1000, 200000), K=rng.randint(1, 4), n_tx=rng.randint(1, 4),
              n_rx=rng.randint(1, 4), C=_logint(rng, 1, 256), S=_logint(rng, 16, 1024))
    if rng.random() < 0.5:
        c["S"] = rng.choice([64, 128, 256, 256, 512])
    if rng.random() < 0.5:
        c["C"] = rng.choice([16, 32, 64, 128])
    big = {"forward": 1448, "step": 1024, "recon": 1024, "batch": 256, "geometry": 1448, "synth": 400,
           "backward": 400}[kind]
    c["nx"], c["ny"] = _logint(rng, 64, big), _logint(rng, 64, big)
    speed = rng.choice([0.0, rng.uniform(0.2, 2.0), rng.uniform(0.2, 2.0), rng.uniform(2.0, 15.0)])
    ang = rng.choice([0.0, 0.0, rng.uniform(-math.pi, math.pi)])
    c["vx"], c["vz"] = round(speed * math.sin(ang), 3), round(speed * math.cos(ang), 3)
    if kind in ("synth", "backward"):
        c["nf"] = min(c["nf"], 8000)   # prepare() traces these by brute force
    if kind == "backward":
        c["materials"], c["attached"] = rng.random() < 0.5, rng.random() < 0.5
    if kind == "step":
        c["materials"] = rng.random() < 0.3
    if kind in ("geometry", "forward", "step"):
        c["shadow"], c["jitter"] = rng.random() < 0.3, rng.random() < 0.3
    if kind == "geometry":
        c["refit"] = rng.random() < 0.5
    if kind == "batch":
        c["n"], c["nf"] = rng.randint(2, 24), min(c["nf"], 20000)
    return c


# ------------------------------------------------------------------ scenes
@functools.lru_cache(maxsize=16)
def _mesh(mesh, nf):
    """(verts float64, faces int32, half-width tangent of the ray grid)."""
    if mesh == "trihedral":
        sc = S.trihedral_plate()
    elif mesh == "icosphere":
        sc = S.icosphere_scene(level=5, jitter=0.0)
    elif mesh == "clutter":
        sc = S.clutter_scene()
    elif mesh == "imaging":
        sc = S.imaging_scene()
    elif mesh == "geodesic":
        sc = S.recon_scenes()[0]
    else:
        n_lat = max(3, int(round(math.sqrt(nf / 4.0)))) + 1
        v, f = S.superquadric_object(7, 2 * (n_lat - 1), n_lat, (0.3, 0.25, 0.2), (0.0, 0.0, 1.6))
        return v, np.asarray(f, np.int32), S.fov_tan(0.32, 1.6)
    return sc.verts.astype(np.float64), sc.faces, sc.grid.tan_hx


def _scene(case, seed):
    """The case's scene: the object a few millimetres from its nominal place
    (the icosphere with its workload's 2 mm rough surface instead)."""
    v, f, th = _mesh(case["mesh"], case["nf"])
    rng = np.random.default_rng(seed)
    if case["mesh"] == "icosphere":
        v = v + rng.normal(0.0, 2e-3, v.shape)
    else:
        v = v + rng.normal(0.0, 3e-3, 3)
    fc = 62e9 if case["planar"] else 77e9
    vel = (case["vx"], 0.0, case["vz"])
    if case["planar"]:
        radar = S.planar_radar(case["n_tx"], case["n_rx"], fc, vel=vel)
        chirp = S.Chirp(fc=fc, slope=7e9 / 25.6e-6, n_samples=case["S"], n_chirps=case["C"])
    else:
        radar = S.default_radar(case["n_tx"], case["n_rx"], fc, vel=vel)
        chirp = S.Chirp(n_samples=case["S"], n_chirps=case["C"])
    grid = S.Grid(case["nx"], case["ny"], th, th, case["K"], shadow=case["shadow"],
                  jitter_seed=seed if case["jitter"] else None)
    mat_id, mats = None, []
    if case["materials"]:
        mats = [(S.MAT_TE, 4.0, 0.02), (S.MAT_TM, 6.0, 0.1), (S.MAT_PEC, 1.0, 0.0)]
        mat_id = (np.arange(len(f)) * 7 // 11 % 3).astype(np.uint16)
        radar.atten = 0.05
    return S.Scene("case", np.ascontiguousarray(v, np.float32), np.ascontiguousarray(f, np.int32), radar, chirp,
                   grid, mat_id, mats)


def _measured(case, seed, noise=0.02):
    """A measured IF cube [V, C, S]: 24 point scatterers and receiver noise, at
    the level of the simulated ones."""
    g = torch.Generator().manual_seed(int(seed) * 2654435761 % (1 << 31))
    dev, dt = _device(), torch.float64
    V, C, Sn = case["n_tx"] * case["n_rx"], case["C"], case["S"]
    p = torch.rand((24, 5), generator=g, dtype=dt).to(dev)
    amp = 2e-3 * (0.1 + p[:, 0]) * torch.exp(2j * math.pi * p[:, 4])
    ev = torch.exp(2j * math.pi * torch.arange(V, device=dev)[:, None] * (p[:, 1] - 0.5) * 0.6)
    ec = torch.exp(2j * math.pi * torch.arange(C, device=dev)[:, None] * (p[:, 2] - 0.5) * 0.2)
    es = torch.exp(2j * math.pi * torch.arange(Sn, device=dev)[:, None] * (0.03 + 0.2 * p[:, 3]))
    x = torch.einsum("vk,ck,sk->vcs", (ev * amp).cpu(), ec.cpu(), es.cpu())
    n = torch.randn((V, C, Sn, 2), generator=g, dtype=torch.float32).to(dt)
    return (x + 2e-3 * noise * torch.view_as_complex(n)).to(torch.complex64).to(dev)


def _simulator(case, seed, **kw):
    from paper_2311_13182_amd.sbr import Simulator
    return Simulator(_scene(case, seed), _device(), **kw)


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    from paper_2311_13182_amd import sbr as B
    kind = case["kind"]
    st = {"case": case}
    if kind in ("image", "detect"):
        sc = S.single_triangle()
        sc.radar, sc.chirp = S.default_radar(case["n_tx"], case["n_rx"]), S.Chirp(n_samples=case["S"],
                                                                                 n_chirps=case["C"])
        st["sim"] = B.Simulator(sc, _device(), n_angle=case["n_angle"], backward=False)
        st["cube"] = _measured(case, seed, 0.3 if kind == "detect" else 0.02)
        if kind == "image":
            st["H"] = _image64(case, _measured(case, seed + 7919)).abs().square().float().contiguous()
        return st
    if kind == "batch":
        sims = [_simulator(_request(case, i), seed + i, backward=False, cube=False) for i in range(case["n"])]
        st["sims"] = sims
        st["table"] = torch.empty(B.sbr_batch_table_bytes(case["n"]), dtype=torch.uint8, device=_device())
        return st
    sim = st["sim"] = _simulator(case, seed, backward=kind in ("step", "recon", "backward"),
                                 cube=kind == "recon" or bool(case.get("image")))
    if kind == "step":
        st["target"] = _measured(case, seed + 7919)
    elif kind == "recon":
        st["verts"] = sim.mesh.verts.clone().requires_grad_(True)
        st["H"] = _image64(case, _measured(case, seed + 7919)).abs().square().float().contiguous()
        st["scale"] = 1.0 / float(st["H"].double().square().mean())
        sim.build()
    elif kind == "geometry":
        sim.build()
    elif kind in ("synth", "backward"):
        h = _trace64(sim.scene)
        sim.hits = B.Hits(h["tri"].int().contiguous(), h["t"].float().contiguous(), h["u"].float().contiguous(),
                          h["v"].float().contiguous(), h["flags"].to(torch.uint8).contiguous())
        if kind == "backward":
            st["grad_if"] = _measured(case, seed + 7919)
    return st


def _request(case, i):
    """Request i of a batch: mesh size, antennas and chirps vary as in the
    serving mix."""
    return dict(case, nf=max(1000, int(case["nf"] * (i % 5 + 1) / 5)), n_tx=1 + i % 3,
                C=max(1, case["C"] >> (i % 2)), K=2 + i % 3 if case["K"] > 1 else 1)


# ------------------------------------------------------------------ run
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "batch":
        from paper_2311_13182_amd import sbr as B
        items, cubes = [], []
        for sim in st["sims"]:
            sim.build()
            sim.trace()
            cubes.append(torch.empty((sim.V, sim.C, sim.S, 2), dtype=torch.float32, device=sim.device))
            items.append((sim.mesh, sim.scene.radar, sim.scene.grid, sim.hits, sim.scene.chirp, sim.flags,
                          cubes[-1], sim.scratch))
        B.sbr_synth_if_batched(items, st["table"])
        return {"cubes": cubes}
    sim = st["sim"]
    if kind == "forward":
        sim.build()
        return {"cube": sim.forward()}
    if kind == "step":
        sim.build()
        cube = sim.forward()
        out = {"cube": cube}
        if case.get("image"):
            out["image"] = sim.radar_cube(cube)
        grad, out["loss"] = sim.loss_grad(cube, st["target"])
        out["verts"] = sim.backward(grad, reuse_paths=True)
        return out
    if kind == "recon":
        from paper_2311_13182_amd.autograd import HeatmapLoss, RadarCubeFunction, simulate
        st["verts"].grad = None
        cube = simulate(st["verts"], sim)
        loss = HeatmapLoss.apply(RadarCubeFunction.apply(cube, sim, 0), st["H"], sim, st["scale"])
        loss.backward()
        return {"cube": cube, "loss": loss, "verts": st["verts"].grad}
    if kind == "geometry":
        sim.build(refit=case["refit"])
        h = sim.trace()
        return {"tri": h.tri, "t": h.t, "u": h.u, "v": h.v, "flags": h.flags}
    if kind == "synth":
        return {"cube": sim.synth()}
    if kind == "backward":
        dev, n = sim.device, len(sim.mesh.materials)
        gm = torch.zeros((n, 2), device=dev) if n else None
        gr, gR, ga = torch.zeros(6, device=dev), torch.zeros((3, 3), device=dev), torch.zeros(1, device=dev)
        gv = sim.backward(st["grad_if"], None, gm, gr, gR, attached=case["attached"], grad_atten=ga)
        return {"verts": gv, "radar": gr, "rot": gR, "atten": ga, "materials": gm}
    if kind == "image":
        X = sim.radar_cube(st["cube"], window=case["window"])
        grad, loss = sim.loss_grad(X, st["H"], mode=1)
        return {"image": X, "loss": loss, "grad": sim.radar_cube(grad, direction=1, window=case["window"])}
    X = sim.radar_cube(st["cube"], window=case["window"])
    det, _, n = sim.cfar(X, max_points=4096)
    return {"image": X, "n": n, "cloud": sim.cloud(det, n)}


# ------------------------------------------------------------------ work
def work(case):
    """Bytes: inputs once in, outputs once out.  Operations: a box test per tree
    level and a few triangle tests per closest-hit query, about 300 per path
    for its geometry, 60 per path and antenna for its phase and 7 complex
    grid taps for its share of the sum (the least any gridding form needs,
    both ways with a backward pass), 5 N log2 N per transform."""
    kind = case["kind"]
    V, C, Sn = case["n_tx"] * case["n_rx"], case["C"], case["S"]
    if kind == "batch":
        parts = [work(dict(_request(case, i), kind="forward")) for i in range(case["n"])]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    cube = 8.0 * V * C * Sn
    if kind in ("image", "detect"):
        na = max(case["n_angle"], V)
        fft = 5.0 * V * C * Sn * math.log2(max(2, C * Sn)) + 5.0 * na * C * Sn * math.log2(na)
        if kind == "detect":
            return {"bytes": cube + na * C * Sn * 8.0 + 4096 * 16, "flops": fft + 3.0 * na * C * Sn}
        return {"bytes": 2 * cube + na * C * Sn * (8.0 + 4.0), "flops": 2 * fft + 10.0 * na * C * Sn}
    R, K, nf = case["nx"] * case["ny"], case["K"], max(2, case["nf"])
    if case["mesh"] == "imaging":
        nf = 20012
    paths = 0.4 * R * K
    mesh = 6.0 * nf + 12.0 * nf
    trace = 0.6 * R * K * (14.0 * math.log2(nf) + 3 * 27.0) * (2 if case["shadow"] else 1)
    synth = paths * (300.0 + V * (60.0 + 7 * 4.0)) + 10.0 * V * C * Sn * math.log2(2 * Sn)
    back = 2.0 * paths * (300.0 + V * (60.0 + 7 * 8.0)) + 20.0 * V * C * Sn * math.log2(2 * Sn)
    image = 0.0
    hits = 17.0 * R * K
    if kind == "recon" or case.get("image"):
        na = 64 * 64 if case["planar"] else max(64, V)
        image = 8.0 * na * C * Sn
    if kind == "geometry":
        return {"bytes": mesh + hits, "flops": trace}
    if kind == "synth":
        return {"bytes": mesh + 5.0 * R * K + cube, "flops": synth}
    if kind == "backward":
        return {"bytes": 2 * mesh + 5.0 * R * K + cube, "flops": back}
    if kind == "forward":
        return {"bytes": mesh + cube, "flops": trace + synth}
    return {"bytes": 2 * mesh + 2 * cube + image, "flops": trace + synth + back}


# ------------------------------------------------------------------ exact
def _image64(case, cube, window=0):
    """Range, Doppler and angle DFTs in 64 bits: [V,C,S] -> [Na,C,S]."""
    x = cube.to(torch.complex128)
    V, C, Sn = x.shape
    if window:
        x = x * _hann(C, x.device)[None, :, None] * _hann(Sn, x.device)[None, None, :]
    na = max(case.get("n_angle", 64), V)
    return torch.fft.fft(torch.fft.fft2(x), n=na, dim=0)


def _image64_adjoint(X, V, window=0):
    na, C, Sn = X.shape
    x = torch.fft.ifft(torch.fft.ifft2(X, norm="forward"), dim=0, norm="forward")[:V]
    if window:
        x = x * _hann(C, x.device)[None, :, None] * _hann(Sn, x.device)[None, None, :]
    return x


def _hann(n, dev):
    if n == 1:
        return torch.ones(1, dtype=torch.float64, device=dev)
    return 0.5 - 0.5 * torch.cos(2 * math.pi * torch.arange(n, dtype=torch.float64, device=dev) / (n - 1))


def _philox_pair(n, seed, dev):
    """Philox-4x32-10 words 0 and 1 at counters (0..n-1, 0, 0, 0), as uniforms."""
    m32 = 0xFFFFFFFF
    c0 = torch.arange(n, dtype=torch.int64, device=dev)
    c1 = torch.zeros_like(c0)
    c2, c3 = c1.clone(), c1.clone()
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57   # wrap modulo 2^64: the words are right
        h0, l0 = (p0 >> 32) & m32, p0 & m32
        h1, l1 = (p1 >> 32) & m32, p1 & m32
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return (c0 >> 8).double() / 16777216.0, (c1 >> 8).double() / 16777216.0


def _rays64(sc, rot):
    """Unit directions [R,3] in the world frame, radar-frame directions and the
    cells' solid angles of the ray grid."""
    g, dev = sc.grid, rot.device
    r = torch.arange(g.nx * g.ny, device=dev)
    jx = jy = 0.5
    if g.jitter_seed is not None:
        jx, jy = _philox_pair(g.nx * g.ny, int(g.jitter_seed), dev)
    u = g.tan_hx * (2.0 * ((r % g.nx).double() + jx) / g.nx - 1.0)
    v = g.tan_hy * (2.0 * ((r // g.nx).double() + jy) / g.ny - 1.0)
    q = 1.0 + u * u + v * v
    loc = torch.stack([u, v, torch.ones_like(u)], 1) / q.sqrt()[:, None]
    return loc @ rot.T, (2 * g.tan_hx / g.nx) * (2 * g.tan_hy / g.ny) / q ** 1.5


def _closest(o, d, prev, va, e1, e2, tmin, tmax=None):
    """Closest hit of rays (o, d) over all triangles in 64 bits: t1, t2, face
    (-1: none); with tmax, whether any hit lies in (tmin, tmax)."""
    N = torch.linalg.cross(e1, e2)
    uf = torch.cat([e2, -torch.linalg.cross(e2, va)], 1).T
    vf = torch.cat([-e1, -torch.linalg.cross(va, e1)], 1).T
    aN = (va * N).sum(1)
    n, nf = len(o), len(va)
    step = max(1, (1 << 26) // nf)
    inf = torch.inf
    t1s, t2s, fs, any_ = [], [], [], []
    for b in range(0, n, step):
        oo, dd = o[b:b + step], d[b:b + step]
        md = torch.cat([torch.linalg.cross(oo, dd), dd], 1)
        det = -(dd @ N.T)
        u, v = (md @ uf) / det, (md @ vf) / det
        ok = (u >= 0) & (v >= 0) & (u + v <= 1)
        del u, v
        t = (oo @ N.T - aN) / det
        ok &= (t > tmin) & torch.isfinite(t)
        if prev is not None:
            ok[torch.arange(len(oo), device=o.device), prev[b:b + step].clamp(min=0)] &= prev[b:b + step] < 0
        if tmax is not None:
            any_.append((ok & (t < tmax[b:b + step, None])).any(1))
            continue
        t = torch.where(ok, t, inf)
        t1, f = t.min(1)
        t.scatter_(1, f[:, None], inf)
        t1s.append(t1)
        t2s.append(t.min(1)[0])
        fs.append(torch.where(torch.isfinite(t1), f, -1))
    if tmax is not None:
        return torch.cat(any_)
    return torch.cat(t1s), torch.cat(t2s), torch.cat(fs)


def _trace64(sc):
    """Closest-hit records [K, R] and their flags, every triangle tested."""
    dev = _device()
    va, e1, e2, _ = _triangles(sc, torch.as_tensor(sc.verts, device=dev).double())
    rot = torch.as_tensor(np.asarray(sc.radar.rot), device=dev).double()
    org = torch.as_tensor(np.asarray(sc.radar.origin), device=dev).double()
    d, _ = _rays64(sc, rot)
    R, K = len(d), sc.grid.max_bounces
    out = {k: torch.zeros((K, R), dtype=torch.float64, device=dev) for k in ("t", "u", "v")}
    tri = torch.full((K, R), -1, dtype=torch.int64, device=dev)
    flags = torch.zeros((K, R), dtype=torch.int64, device=dev)
    idx = torch.arange(R, device=dev)
    o, prev, L, anc = org.expand(R, 3), None, torch.zeros(R, dtype=torch.float64, device=dev), \
        torch.zeros(R, dtype=torch.bool, device=dev)
    for k in range(K):
        t1, t2, f = _closest(o, d, prev, va, e1, e2, sc.grid.t_min)
        hit = f >= 0
        idx, o, d, L, anc, t1, t2, f = (x[hit] for x in (idx, o, d, L, anc, t1, t2, f))
        if len(idx) == 0:
            break
        a, p, q = va[f], e1[f], e2[f]
        N = torch.linalg.cross(p, q)
        nl = N.norm(dim=1)
        x = o + t1[:, None] * d
        w = x - a
        b1 = (torch.linalg.cross(w, q) * N).sum(1) / nl ** 2
        b2 = (torch.linalg.cross(p, w) * N).sum(1) / nl ** 2
        dn = (d * N).sum(1) / nl
        L = L + t1
        delta = 1e-6 * L.clamp(min=1.0)
        de = torch.minimum((1 - b1 - b2).abs() * nl / (q - p).norm(dim=1),
                           torch.minimum(b1.abs() * nl / q.norm(dim=1), b2.abs() * nl / p.norm(dim=1)))
        fl = 16 * anc + 1 * (de < delta) + 2 * (t2 - t1 < delta) + 4 * (dn.abs() < 1e-6) + \
            8 * (t1 < 2 * sc.grid.t_min)
        anc = anc | (fl > 0)
        if sc.grid.shadow and k > 0:
            s = org - x
            D = s.norm(dim=1)
            fl = fl + 32 * _closest(x, s / D[:, None], f, va, e1, e2, sc.grid.t_min, D - sc.grid.t_min)
        tri[k, idx], flags[k, idx] = f, fl
        out["t"][k, idx], out["u"][k, idx], out["v"][k, idx] = t1, b1, b2
        d = d - 2 * dn[:, None] * N / nl[:, None]
        o, prev = x, f
    return dict(out, tri=tri, flags=flags)


def _triangles(sc, verts):
    f = torch.as_tensor(sc.faces, device=verts.device).long()
    a = verts[f[:, 0]]
    return a, verts[f[:, 1]] - a, verts[f[:, 2]] - a, f


def _fresnel64(mode, eps_r, sigma, ci, fc):
    eps = torch.complex(eps_r, -sigma / (2 * math.pi * fc * EPS0))
    n = eps.sqrt()
    ct = (1 - (1 - ci * ci) / eps).sqrt()
    te, tm = (ci - n * ct) / (ci + n * ct), (n * ci - ct) / (n * ci + ct)
    return torch.where(mode == 1, te, torch.where(mode == 2, tm, torch.full_like(te, -1.0)))


def _paths64(sc, h, par, attached=False):
    """Differentiable path records from frozen hit records: amplitude [P]
    complex, delay [V, P], delay rate [P].  par: verts, origin, velocity, rot,
    atten, materials [n, 2] as 64-bit tensors.  attached: samples follow their
    first hit (fixed barycentrics, cell weight times D / D0)."""
    dev = par["verts"].device
    va, e1, e2, _ = _triangles(sc, par["verts"])
    org, rd = par["origin"], sc.radar
    txl = torch.as_tensor(np.asarray(rd.tx), device=dev).double()
    rxl = torch.as_tensor(np.asarray(rd.rx), device=dev).double()
    tx, rx = org + txl @ par["rot"].T, org + rxl @ par["rot"].T
    d, dw = _rays64(sc, par["rot"])
    tri, flags = h["tri"], h["flags"]
    mode = mat = None
    if sc.mat_id is not None:
        mat = torch.as_tensor(sc.mat_id.astype(np.int64), device=dev)
        mode = torch.as_tensor([m[0] for m in sc.materials], device=dev)
    idx = torch.arange(tri.shape[1], device=dev)
    o, L, Lmid = org.expand(len(idx), 3), 0.0, 0.0
    pr = torch.ones(len(idx), dtype=torch.complex128, device=dev)
    alive = torch.ones(len(idx), dtype=torch.bool, device=dev)
    amps, taus, rates = [], [], []
    x1 = d1 = None
    for k in range(tri.shape[0]):
        keep = tri[k, idx] >= 0
        idx, o, d, dw, pr, alive = (z[keep] for z in (idx, o, d, dw, pr, alive))
        if k:
            L, Lmid, x1, d1 = L[keep], Lmid[keep], x1[keep], d1[keep]
        if len(idx) == 0:
            break
        f = tri[k, idx]
        a, p, q = va[f], e1[f], e2[f]
        N = torch.linalg.cross(p, q)
        nl = N.norm(dim=1)
        if k == 0 and attached:
            with torch.no_grad():
                x = o + (((a - o) * N).sum(1) / (d * N).sum(1))[:, None] * d
                w = x - a
                b1 = (torch.linalg.cross(w, q) * N).sum(1) / nl ** 2
                b2 = (torch.linalg.cross(p, w) * N).sum(1) / nl ** 2
            x = a + b1[:, None] * p + b2[:, None] * q
            r0 = (x - o).norm(dim=1)
            D = (N * (x - o)).sum(1).abs() / r0 ** 3
            dw = dw * D / D.detach()
            d = (x - o) / r0[:, None]
        else:
            x = o + (((a - o) * N).sum(1) / (d * N).sum(1))[:, None] * d
        dn = (d * N).sum(1) / nl
        ci = dn.abs()
        if mat is None:
            pr = -pr
        else:
            m = mat[f]
            pr = pr * _fresnel64(mode[m], par["materials"][m, 0], par["materials"][m, 1], ci, sc.chirp.fc)
        seg = (x - o).norm(dim=1)
        L = L + seg
        Lmid = Lmid + seg if k else torch.zeros_like(seg)
        if k == 0:
            x1, d1 = x, d
        alive = alive & ((flags[k, idx] & ~32) == 0)
        out = alive & ((flags[k, idx] & 32) == 0)
        xo, Rk = x[out], (x[out] - org).norm(dim=1)
        A = pr[out] * (dw[out] * ci[out] / (L[out] * Rk) * torch.exp(-par["atten"] * (L[out] + Rk)))
        dt = (x1[out][None] - tx[:, None]).norm(dim=2)
        dr = (xo[None] - rx[:, None]).norm(dim=2)
        tau = (dt[:, None] + dr[None, :] + Lmid[out]) / C0
        amps.append(A)
        taus.append(tau.reshape(-1, int(out.sum())))
        rates.append(2 * (d1[out] @ par["velocity"]) / C0)
        d = d - 2 * dn[:, None] * N / nl[:, None]
        o = x
    return torch.cat(amps), torch.cat(taus, 1), torch.cat(rates)


def _factors64(sc, A, tau, rate):
    """Eq. 8 around the middle chirp and sample: per antenna the factors
    U [P, C], W [P, S] of the phase, the amplitude they multiply, and the
    terms of e^{2 pi j c' s' eps} (a short series)."""
    ch, dev = sc.chirp, A.device
    c = torch.arange(ch.n_chirps, device=dev).double()
    s = torch.arange(ch.n_samples, device=dev).double()
    cm, sm = (ch.n_chirps - 1) / 2.0, (ch.n_samples - 1) / 2.0
    nu = ch.fc * ch.t_chirp * rate
    gam, eps = ch.slope / ch.fs * tau, ch.slope / ch.fs * ch.t_chirp * rate
    tp = 2 * math.pi

    def cis(x):
        x = tp * (x - torch.round(x))
        return torch.complex(torch.cos(x), torch.sin(x))

    U = cis(c[None] * (nu + sm * eps)[:, None])
    amp = A * cis(ch.fc * tau) * cis(-cm * sm * eps)
    W = cis(s[None] * (gam + cm * eps)[:, None])
    z = tp * eps * max(cm, 0.5) * max(sm, 0.5)
    n, term, big = 1, 1.0, float(z.abs().max()) if len(z) else 0.0
    while term > 1e-13:
        term *= big / n
        n += 1
    return U, W, amp, z, (c - cm) / max(cm, 0.5), (s - sm) / max(sm, 0.5), n


def _synth64(sc, A, tau, rate, chunk=1 << 16):
    V, C, Sn = tau.shape[0], sc.chirp.n_chirps, sc.chirp.n_samples
    out = torch.zeros((V, C, Sn), dtype=torch.complex128, device=A.device)
    for b in range(0, len(A), chunk):
        e = slice(b, b + chunk)
        for v in range(V):
            U, W, amp, z, c1, s1, n = _factors64(sc, A[e], tau[v, e], rate[e])
            f = 1.0
            for k in range(n):
                T = (U * amp[:, None]).T @ W
                out[v] += T * (c1[:, None] * s1[None, :]) ** k / f
                amp = amp * (1j * z)
                f *= k + 1
    return out


def _adjoint64(sc, A, tau, rate, G, chunk=1 << 16):
    """dL/dA (complex), dL/dtau [V, P], dL/drate [P] of Re sum conj(G) dS."""
    ch, V = sc.chirp, tau.shape[0]
    dev = A.device
    s = torch.arange(ch.n_samples, device=dev).double()
    c = torch.arange(ch.n_chirps, device=dev).double()
    w2 = ch.fc + ch.slope / ch.fs * s
    gA, gtau, grate = torch.zeros_like(A), torch.zeros_like(tau), torch.zeros_like(rate)
    for b in range(0, len(A), chunk):
        e = slice(b, b + chunk)
        for v in range(V):
            U, W, z0, z, c1, s1, n = _factors64(sc, torch.ones_like(A[e]), tau[v, e], rate[e])
            X = G[v].conj()
            P = Q = T = 0.0
            f = 1.0
            zk = z0
            for k in range(n):
                Ws = W * s1[None] ** k
                Y = (U * c1[None] ** k) @ X
                P = P + (Ws * Y).sum(1) * zk / f
                Q = Q + (Ws * Y * w2[None]).sum(1) * zk / f
                Y = (U * (c1 ** k * c * ch.t_chirp)[None]) @ X
                T = T + (Ws * Y * w2[None]).sum(1) * zk / f
                zk = zk * (1j * z)
                f *= k + 1
            gA[e] += P.conj()
            gtau[v, e] = -2 * math.pi * (A[e] * Q).imag
            grate[e] += -2 * math.pi * (A[e] * T).imag
    return gA, gtau, grate


def _parameters(sc):
    dev = _device()

    def t(x):
        return torch.as_tensor(np.asarray(x, np.float64), device=dev).clone().requires_grad_(True)

    return {"verts": t(sc.verts), "origin": t(sc.radar.origin), "velocity": t(sc.radar.vel), "rot": t(sc.radar.rot),
            "atten": t(sc.radar.atten), "materials": t([m[1:] for m in sc.materials] or np.zeros((0, 2)))}


def _backward64(sc, A, tau, rate, G, par, attached=False):
    gA, gtau, grate = _adjoint64(sc, A.detach(), tau.detach(), rate.detach(), G)
    total = (gA.conj() * A).real.sum() + (gtau * tau).sum() + (grate * rate).sum()
    keys = list(par)
    return dict(zip(keys, torch.autograd.grad(total, [par[k] for k in keys], allow_unused=True)))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("image", "detect"):
        V = case["n_tx"] * case["n_rx"]
        X = _image64(case, _measured(case, seed, 0.3 if kind == "detect" else 0.02), case["window"])
        if kind == "detect":
            return {"image": X, "n": None, "cloud": None}
        H = _image64(case, _measured(case, seed + 7919)).abs().square().float().double()
        q = X.abs().square() - H
        return {"image": X, "loss": q.square().mean().reshape(1),
                "grad": _image64_adjoint(4 * q * X / X.numel(), V, case["window"])}
    if kind == "batch":
        parts = [exact(dict(_request(case, i), kind="forward"), seed + i) for i in range(case["n"])]
        return None if any(p is None for p in parts) else {"cubes": [p["cube"] for p in parts]}
    R, K, V = case["nx"] * case["ny"], case["K"], case["n_tx"] * case["n_rx"]
    if R * K * case["nf"] > 2e10 or R * K * V * case["S"] * (1 + case["C"] / 64) > 4e10 or kind == "geometry":
        return None
    sc = _scene(case, seed)
    par = _parameters(sc)
    h = _trace64(sc)
    with torch.set_grad_enabled(kind in ("step", "recon", "backward")):
        A, tau, rate = _paths64(sc, h, par, case["attached"])
    if kind == "backward":
        G = _measured(case, seed + 7919).to(torch.complex128)
        g = _backward64(sc, A, tau, rate, G, par, case["attached"])
        still = np.zeros(3)
        vel = g["velocity"] if g["velocity"] is not None else torch.as_tensor(still, device=A.device)
        return {"verts": g["verts"], "radar": torch.cat([g["origin"], vel]), "rot": g["rot"],
                "atten": g["atten"].reshape(1), "materials": g["materials"] if case["materials"] else None}
    cube = _synth64(sc, A.detach(), tau.detach(), rate.detach())
    if kind in ("forward", "synth"):
        return {"cube": cube}
    out = {"cube": cube}
    if kind == "step":
        if case.get("image"):
            out["image"] = None if case["planar"] else _image64(case, cube)
        D = cube - _measured(case, seed + 7919).to(torch.complex128)
        out["loss"] = D.abs().square().sum().reshape(1)
        G = 2 * D
    else:
        H = _image64(case, _measured(case, seed + 7919)).abs().square().float().double()
        scale = 1.0 / float(H.square().mean())
        X = _image64(case, cube)
        q = X.abs().square() - H
        out["loss"] = q.square().mean() * scale
        G = _image64_adjoint(4 * q * X / X.numel(), V) * scale
    out["verts"] = _backward64(sc, A, tau, rate, G, par)["verts"]
    return out
