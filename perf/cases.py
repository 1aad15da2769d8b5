"""The workloads that the framework's speed is measured on, as a program of a user runs them.

Every case is one call, or the few calls that belong together, through the public entry points:

  pose    et.simulate: trace a pose and synthesise its spectra (optionally keeping the paths)
  frame   Scene.refit to moved vertices, then et.simulate: one frame of an animated scene
  batch   Batch.run: many poses over several scenes, forward and adjoint
  synth   et.synthesize: spectra of records that are given
  fit     SpectraFn forward and backward: one step of fitting material coefficients and receiver
          positions to measured spectra
  build   Scene: the tree and the curvature of a mesh
  signal  et.impulse_response and et.receiver_signal of given spectra

Sizes follow the repository's own workloads (wall and sphere, room with a 32-microphone array,
foliage, pose batches) and the range around them, odd and ragged sizes among them.  All inputs
are synthetic and made from the seed.  Whole poses have no 64-bit value: which triangle a ray near
an edge hits is decided in FP32, so a 64-bit trace would follow other paths for some rays.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2602_19652_amd as et

C_SOUND = 343.0
A1 = 3.5e-5          # dB / (m Hz)
SENSOR = (1.0, 4.0, 1.2)


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest call: a wall and a sphere, one emitter, two receivers; latency and launches
        dict(name="pose tiny", kind="pose", scene="wall", objects=1, rays=16384, bounces=3, mics=2, bins=1024,
             bands=8, diff=0, per_mesh=False, passive=False, directivity=False, product=False, per_rx=False,
             records=True),
        # the main workload: an office with a 32-microphone array, diffraction included
        dict(name="pose room", kind="pose", scene="room", objects=200, rays=1 << 20, bounces=4, mics=32, bins=4096,
             bands=8, diff=65536, per_mesh=False, passive=False, directivity=False, product=False, per_rx=False,
             records=False),
        # a million triangles of leaves, two ears with a directivity table, many bins
        dict(name="pose foliage", kind="pose", scene="foliage", objects=62500, rays=1 << 20, bounces=6, mics=2,
             bins=8192, bands=8, diff=0, per_mesh=False, passive=False, directivity=True, product=False,
             per_rx=False, records=True),
        # ragged sizes and the options together: candidates per mesh, direct paths, paths kept
        dict(name="pose ragged", kind="pose", scene="room", objects=61, rays=50003, bounces=3, mics=7, bins=1000,
             bands=5, diff=257, per_mesh=True, passive=True, directivity=False, product=False, per_rx=False,
             records=True),
        # an animated scene: objects moved between frames, line of sight per receiver
        dict(name="frame room", kind="frame", scene="room", objects=200, rays=1 << 15, bounces=3, mics=8, bins=2048,
             bands=8, diff=8192, per_mesh=False, passive=False, directivity=False, product=False, per_rx=True,
             records=False),
        # poses of a trajectory and of other scenes in one call, with gradients for each
        dict(name="batch poses", kind="batch", jobs=24, scenes=5, objects=60, rays=1 << 16, bounces=4, mics=8,
             bins=2048, bands=8, adjoint=True),
        # synthesis alone over stored paths, the array's size
        dict(name="synth array", kind="synth", records=250000, mics=32, bins=4096, bands=8, materials=16,
             directivity=False),
        # synthesis with a bin count off any power of two and bands of unequal width
        dict(name="synth ragged", kind="synth", records=60000, mics=6, bins=3000, bands=7, materials=5,
             directivity=False),
        # a fitting step at the batch's bins
        dict(name="fit array", kind="fit", records=100000, mics=16, bins=2048, bands=8, materials=16,
             directivity=False),
        # a small fitting step with ragged bins
        dict(name="fit ragged", kind="fit", records=20011, mics=4, bins=1500, bands=6, materials=9,
             directivity=False),
        # the scene of the main workload, built
        dict(name="build room", kind="build", scene="room", objects=200),
        # the time domain of the main workload's spectra: responses at 320 kHz and a 2 ms call
        dict(name="signal array", kind="signal", mics=32, bins=4096, samples=16384, call=640),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _bins(rng, lo, hi):
    """Bins: half of the draws a multiple of 64, the others any number."""
    F = _log(rng, lo, hi)
    return F if rng.random() < 0.5 else max(64, F // 64 * 64)


def draw(rng):
    kind = rng.choice(["pose", "pose", "pose", "frame", "batch", "synth", "synth", "fit", "fit", "build", "signal"])
    if kind in ("pose", "frame"):
        scene = rng.choice(["wall", "room", "room", "foliage"]) if kind == "pose" else "room"
        c = dict(kind=kind, scene=scene, objects=1, rays=_log(rng, 1 << 12, 1 << 20), bounces=rng.randint(1, 6),
                 mics=_log(rng, 1, 32), bins=_bins(rng, 200, 4096), bands=rng.choice([1, 3, 5, 8, 8, 10]), diff=0,
                 per_mesh=False, passive=rng.random() < 0.3, directivity=False, product=rng.random() < 0.15,
                 per_rx=False, records=rng.random() < 0.3)
        if scene == "room":
            c["objects"] = _log(rng, 10, 200)
            if rng.random() < 0.5:
                c["per_mesh"] = rng.random() < 0.3
                c["diff"] = _log(rng, 64, 512) if c["per_mesh"] else _log(rng, 1000, 65536)
            c["per_rx"] = kind == "frame" and rng.random() < 0.5
        if scene == "foliage":
            c.update(objects=_log(rng, 2000, 62500), mics=rng.randint(1, 2), directivity=rng.random() < 0.7,
                     bins=_bins(rng, 1000, 8192), product=False)
        if kind == "frame":
            c.update(rays=_log(rng, 1 << 12, 1 << 17), product=False)
        while c["rays"] * c["bounces"] * c["mics"] * c["bins"] > (1 << 36):
            c["rays"] = c["rays"] * 3 // 4
        if c["per_rx"]:
            c["rays"] = max(2048, min(c["rays"], (1 << 18) // c["mics"]))
        return c
    if kind == "batch":
        c = dict(kind=kind, jobs=_log(rng, 3, 24), scenes=rng.randint(1, 6), objects=_log(rng, 10, 60),
                 rays=_log(rng, 1 << 12, 1 << 16), bounces=rng.randint(2, 4), mics=_log(rng, 1, 8),
                 bins=_bins(rng, 256, 2048), bands=rng.choice([4, 8]), adjoint=rng.random() < 0.7)
        while c["jobs"] * c["rays"] * c["mics"] * c["bins"] > (1 << 33):
            c["rays"] = c["rays"] * 3 // 4
        return c
    if kind in ("synth", "fit"):
        c = dict(kind=kind, records=_log(rng, 1000, 250000), mics=_log(rng, 1, 32), bins=_bins(rng, 200, 4096),
                 bands=rng.choice([1, 4, 6, 7, 8, 8, 16]), materials=rng.randint(1, 16),
                 directivity=kind == "synth" and rng.random() < 0.3)
        if kind == "fit":   # (an array: its places and materials from enough paths to tell them apart)
            c.update(mics=_log(rng, 4, 32), records=_log(rng, 5000, 250000))
        while c["records"] * c["mics"] * c["bins"] > (1 << 32):
            c["records"] = c["records"] * 3 // 4
        return c
    if kind == "build":
        return dict(kind=kind, scene="room", objects=_log(rng, 5, 200))
    bins = _log(rng, 256, 4096)
    samples = 1 << rng.randint(max(bins - 1, 1).bit_length(), 15)
    return dict(kind=kind, mics=_log(rng, 1, 32), bins=bins, samples=samples, call=_log(rng, 32, 4096))


# ------------------------------------------------------------------ meshes

def _box_template(n):
    """Surface of the unit box, each face n x n quads, shared vertices once."""
    g = np.arange(n + 1)
    lat, quads = {}, []
    for a in range(3):
        u, v = [x for x in range(3) if x != a]
        for side in (0, n):
            for i in range(n):
                for j in range(n):
                    q = []
                    for ii, jj in ((i, j), (i + 1, j), (i + 1, j + 1), (i, j + 1)):
                        c = [0, 0, 0]
                        c[a], c[u], c[v] = side, g[ii], g[jj]
                        q.append(lat.setdefault(tuple(int(x) for x in c), len(lat)))
                    quads.append(q if (side == n) == (a != 1) else q[::-1])
    q = np.array(quads)
    verts = np.array(list(lat), float) / n
    return verts, np.concatenate([q[:, [0, 1, 2]], q[:, [0, 2, 3]]], 1).reshape(-1, 3)


def _cylinder_template(segments, rings):
    ang = 2 * math.pi * np.arange(segments) / segments
    side = np.stack([np.tile(np.cos(ang), rings + 1), np.tile(np.sin(ang), rings + 1),
                     np.repeat(np.arange(rings + 1) / rings, segments)], 1)
    verts = np.vstack([side, [[0, 0, 0], [0, 0, 1]]])
    r, s = np.meshgrid(np.arange(rings), np.arange(segments), indexing="ij")
    a, b = r * segments + s, r * segments + (s + 1) % segments
    c, d = b + segments, a + segments
    s1 = np.arange(segments)
    s2, top, cb = (s1 + 1) % segments, rings * segments, len(side)
    tris = np.concatenate([np.stack([a, b, c], -1).reshape(-1, 3), np.stack([a, c, d], -1).reshape(-1, 3),
                           np.stack([np.full_like(s1, cb), s2, s1], 1),
                           np.stack([np.full_like(s1, cb + 1), top + s1, top + s2], 1)])
    return verts, tris


def _instances(verts, tris):
    """[n][v][3] instances of one template: vertices, triangles and the instance of each triangle."""
    n, v = verts.shape[:2]
    t = (tris[None] + (np.arange(n) * v)[:, None, None]).reshape(-1, 3)
    return verts.reshape(-1, 3), t, np.repeat(np.arange(n), len(tris))


def _merge(parts):
    """Mesh dict of (vertices, triangles, object of each triangle, material of each object) parts."""
    V, T, O, Q, nv, no = [], [], [], [], 0, 0
    for v, t, o, q in parts:
        V.append(v)
        T.append(t + nv)
        O.append(o + no)
        Q.append(np.asarray(q)[o])
        nv += len(v)
        no += len(q)
    return {"vertices": np.concatenate(V).astype(np.float32), "tris": np.concatenate(T).astype(np.int32),
            "tri_object": np.concatenate(O).astype(np.int32), "tri_material": np.concatenate(Q).astype(np.int32),
            "n_objects": no}


def _room(g, objects, box=9, seg=120, rings=3):
    """10 x 8 x 3 m room with boxes and cylinders on the floor, half of each, clear of the sensor."""
    nb = objects // 2
    nc = objects - nb
    xy = np.zeros((0, 2))
    while len(xy) < objects:
        p = np.stack([g.uniform(0.5, 9.5, 2 * objects), g.uniform(0.5, 7.5, 2 * objects)], 1)
        xy = np.concatenate([xy, p[np.hypot(p[:, 0] - SENSOR[0], p[:, 1] - SENSOR[1]) > 1.8]])
    xy = xy[:objects]
    v, t = _box_template(1)
    parts = [(v * [10.0, 8.0, 3.0], t, np.zeros(len(t), int), [0])]
    mat = 1 + np.arange(objects) % 15
    if nb:
        v, t = _box_template(box)
        size, yaw = g.uniform(0.2, 1.5, (nb, 3)), g.uniform(0, 2 * math.pi, nb)
        p = (v[None] - [0.5, 0.5, 0.0]) * size[:, None]
        c, s = np.cos(yaw)[:, None], np.sin(yaw)[:, None]
        p = np.stack([c * p[..., 0] - s * p[..., 1] + xy[:nb, :1], s * p[..., 0] + c * p[..., 1] + xy[:nb, 1:],
                      p[..., 2] + 0.001], -1)
        parts.append((*_instances(p, t), mat[:nb]))
    if nc:
        v, t = _cylinder_template(seg, rings)
        size = np.stack([*[g.uniform(0.1, 0.5, nc)] * 2, g.uniform(0.3, 2.5, nc)], 1)
        p = v[None] * size[:, None] + np.concatenate([xy[nb:], np.full((nc, 1), 0.001)], 1)[:, None]
        parts.append((*_instances(p, t), mat[nb:]))
    return _merge(parts)


def _foliage(g, leaves):
    """Leaf discs of 16 triangles (radius 1 to 5 cm) in a 4 m cube about the sensor."""
    c = g.uniform(0, 4, (leaves, 3))
    c = np.where(np.linalg.norm(c - 2.0, axis=1, keepdims=True) < 0.25, c + 0.3, c)
    n = g.normal(size=(leaves, 3))
    n /= np.linalg.norm(n, axis=1, keepdims=True)
    e1 = np.cross(n, np.where(np.abs(n[:, :1]) < 0.9, [[1.0, 0, 0]], [[0, 1.0, 0]]))
    e1 /= np.linalg.norm(e1, axis=1, keepdims=True)
    e2 = np.cross(n, e1)
    ang = 2 * math.pi * np.arange(16) / 16
    rim = (np.cos(ang)[None, :, None] * e1[:, None] + np.sin(ang)[None, :, None] * e2[:, None])
    v = np.concatenate([c[:, None], c[:, None] + g.uniform(0.01, 0.05, (leaves, 1, 1)) * rim], 1)
    s = np.arange(16)
    t = np.stack([np.zeros_like(s), 1 + s, 1 + (s + 1) % 16], 1)
    return _merge([(*_instances(v, t), np.arange(leaves) % 16)])


def _wall(g):
    """A 4 x 4 m wall and a tessellated sphere (radius 0.5 m, about 1280 triangles) 3 m away."""
    wall = np.array([[4, -2, -2], [4, 2, -2], [4, 2, 2], [4, -2, 2]], float)
    v, t = _cylinder_template(32, 19)
    el = (v[:, 2] - 0.5) * math.pi * 0.98
    el[-2:] = [-math.pi / 2, math.pi / 2]
    ball = 0.5 * np.stack([np.cos(el) * v[:, 0], np.cos(el) * v[:, 1], np.sin(el)], 1)
    a = g.uniform(0.2, 0.3)
    return _merge([(wall, np.array([[0, 1, 2], [0, 2, 3]]), np.zeros(2, int), [0]),
                   (ball + 3 * np.array([math.cos(a), math.sin(a), 0.0]), t, np.zeros(len(t), int), [0])])


def _mesh(case, g):
    if case["scene"] == "wall":
        return _wall(g)
    return _foliage(g, case["objects"]) if case["scene"] == "foliage" else _room(g, case["objects"])


def _area_ref(mesh):
    v, t = mesh["vertices"].astype(np.float64), mesh["tris"]
    return float(np.median(0.5 * np.linalg.norm(np.cross(v[t[:, 1]] - v[t[:, 0]], v[t[:, 2]] - v[t[:, 0]]), axis=1)))


# ------------------------------------------------------------------ poses

def _cone(seed, n, half_angle):
    """n directions on the GPU, uniform over the solid angle of a cone about +x."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.rand(2, n, dtype=torch.float64, device="cuda", generator=g)
    ct = 1.0 - u[0] * (1.0 - math.cos(half_angle))
    st, ph = torch.sqrt(torch.clamp(1 - ct * ct, min=0.0)), 2 * math.pi * u[1]
    return torch.stack([ct, st * torch.cos(ph), st * torch.sin(ph)], 1).float().contiguous()


def _tables(g, q, b):
    return (g.uniform(0.3, 0.99, (q, b)).astype(np.float32), g.uniform(0.05, 0.3, (q, b)).astype(np.float32),
            g.uniform(0.05, 0.3, (q, b)).astype(np.float32))


def _disc(g, m, centre):
    r, a = 0.06 * np.sqrt(g.uniform(0, 1, m)), g.uniform(0, 2 * math.pi, m)
    return np.asarray(centre, float) + np.stack([np.zeros(m), r * np.cos(a), r * np.sin(a)], 1)


def _directivity(g, m, Bd=16, El=32, Az=64):
    az = -math.pi + (np.arange(Az) + 0.5) * 2 * math.pi / Az
    el = -math.pi / 2 + (np.arange(El) + 0.5) * math.pi / El
    base = (1 + np.cos(el)[:, None] * np.cos(az)) / 2
    tab = base[None, None] ** (1 + np.arange(Bd) / 2)[None, :, None, None]
    return (tab * (1 + 0.05 * g.uniform(-1, 1, (m, Bd, El, Az)))).astype(np.float32)


def _settings(case, g, pos, rays, q, tables=None):
    k, beta, d = tables or _tables(g, q, case["bands"])
    s = dict(emitter_pos=pos, emitter_rot=np.eye(3), rx_pos=_disc(g, case["mics"], pos),
             rx_rot=np.repeat(np.eye(3)[None], case["mics"], 0), ray_dirs=rays, x_ref=pos,
             max_bounces=case.get("bounces", 1), max_distance=math.inf, t_eps=1e-5, f_lo=20e3, f_hi=100e3,
             F=case["bins"], c=C_SOUND, atm_a0=0.0, atm_a1=A1, spreading_p=2.0, phase_sign=1, refl_k=k,
             lobe_beta=beta, diff_coef=d)
    if case.get("directivity"):
        s["directivity"] = _directivity(g, case["mics"])
    return s


def _pose(case, seed, g, mesh):
    pos = {"wall": (0.0, 0.0, 0.0), "room": SENSOR, "foliage": (2.0, 2.0, 2.0)}[case["scene"]]
    half = {"wall": math.pi / 6, "room": math.pi / 2, "foliage": math.pi / 3}[case["scene"]]
    s = _settings(case, g, np.array(pos), _cone(seed, case["rays"], half), 16)
    s.update(diff_K=case["diff"], diff_seed=seed, diff_per_mesh=case["per_mesh"],
             diff_max_meshes=mesh["n_objects"] if case["per_mesh"] else 1, path_product=case["product"],
             per_rx_visibility=case["per_rx"])
    if case["passive"]:
        s["passive_coef"] = g.uniform(0.5, 1.0, case["bands"]).astype(np.float32)
    return et.Sim(s)


# ------------------------------------------------------------------ records

def _records(case, seed):
    """Paths of a room as a trace leaves them: points about the sensor, 70 % visible, a twentieth from
    diffraction, reflected directions spread about the way to the receivers."""
    g = np.random.default_rng(seed)
    n = case["records"]
    p = g.uniform([0, 0, 0], [10, 8, 3], (n, 3))
    p = np.where(np.linalg.norm(p - SENSOR, axis=1, keepdims=True) < 0.5, p + 1.0, p)
    w = np.asarray(SENSOR) - p
    leg = np.linalg.norm(w, axis=1)
    d = w / leg[:, None] + 0.4 * g.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    kind = (g.random(n) < 0.05).astype(np.uint8)
    d[kind == 1] = 0.0
    rec = dict(p=p, dout=d.astype(np.float32), rtot=leg + g.exponential(6.0, n) * (kind == 0),
               mat=g.integers(0, case["materials"], n).astype(np.int32), vis=(g.random(n) < 0.7).astype(np.uint8),
               kind=kind)
    # (one ray per record: the workspace of a pose is sized by its rays)
    return rec, _settings(case, g, np.array(SENSOR), np.zeros((n, 3), np.float32), case["materials"])


def _target(case, seed):
    """Measured spectra to fit: random, of about the size of the records' own."""
    g = np.random.default_rng(seed + 7)
    s = 0.002 * math.sqrt(case["records"])
    z = g.normal(size=(2, case["mics"], case["bins"])) * s
    return (z[0] + 1j * z[1]).astype(np.complex64)


# ------------------------------------------------------------------ the cases' three functions

def prepare(case, seed):
    g = np.random.default_rng(seed)
    kind = case["kind"]
    ctx = et.Context()
    st = dict(kind=kind, ctx=ctx)
    if kind in ("pose", "frame"):
        mesh = _mesh(case, g)
        st["area"] = _area_ref(mesh)
        st["scene"] = et.Scene(ctx, mesh, area_ref=st["area"])
        sim = st["sim"] = _pose(case, seed, g, mesh)
        st.update(paths=et.Paths(sim.capacity()), ws=et.Workspace(), keep=case["records"],
                  out=torch.empty(sim.M, sim.F, 2, dtype=torch.float32, device="cuda"))
        if kind == "frame":
            # every object but the room itself moves by up to 10 cm
            shift = g.uniform(-0.1, 0.1, (mesh["n_objects"], 3)) * [1, 1, 0]
            shift[0] = 0.0
            obj = np.zeros(len(mesh["vertices"]), int)
            obj[mesh["tris"].reshape(-1)] = np.repeat(mesh["tri_object"], 3)
            st["moved"] = torch.as_tensor((mesh["vertices"] + shift[obj]).astype(np.float32)).cuda()
    elif kind == "batch":
        scenes, poses = [], []
        for k in range(case["scenes"]):
            mesh = _room(g, max(2, case["objects"] // (k + 1)), box=5, seg=40, rings=4)
            scenes.append(et.Scene(ctx, mesh))
        tables = _tables(g, 16, case["bands"])
        for j in range(case["jobs"]):
            pos = np.array(SENSOR) + [0.3 * math.cos(j), 0.3 * math.sin(j), 0.02 * (j % 7)]
            s = _settings(case, g, pos, _cone(seed * 1000 + j, case["rays"], math.pi / 2), 16, tables)
            poses.append((scenes[j % len(scenes)], et.Sim(s, flags=et.ET_SPECULAR)))
        st["batch"] = et.Batch(ctx, poses)
        gen = torch.Generator(device="cuda").manual_seed(seed)
        st["grad"] = 1e-3 * torch.randn(case["jobs"], case["mics"], case["bins"], dtype=torch.complex64,
                                        device="cuda", generator=gen) if case["adjoint"] else None
    elif kind in ("synth", "fit"):
        rec, s = _records(case, seed)
        st.update(paths=et.Paths.from_records(rec), sim=et.Sim(s, flags=et.ET_SPECULAR), ws=et.Workspace())
        sim = st["sim"]
        if kind == "synth":
            st["out"] = torch.empty(sim.M, sim.F, 2, dtype=torch.float32, device="cuda")
        else:
            # parameters of a fit in torch's default type: the coefficients, and offsets of the
            # receivers from their nominal places
            st.update(k=sim.refl_k.clone().requires_grad_(True), place=sim.rx_pos.clone(),
                      shift=torch.zeros(sim.M, 3, device="cuda", requires_grad=True),
                      target=torch.as_tensor(_target(case, seed)).cuda())
    elif kind == "build":
        mesh = _mesh(case, g)
        st["area"] = _area_ref(mesh)
        st["mesh"] = {k: torch.as_tensor(v).cuda() if isinstance(v, np.ndarray) else v for k, v in mesh.items()}
    else:
        H, call, sim = _spectra(case, seed)
        st.update(H=torch.as_tensor(H).cuda(), call=torch.as_tensor(call).cuda(), n_t=case["samples"], ws=et.Workspace(),
                  ws2=et.Workspace(), sim=et.Sim(sim, flags=et.ET_SPECULAR))
    return st


def run(st):
    kind, ctx = st["kind"], st["ctx"]
    if kind in ("pose", "frame"):
        if kind == "frame":
            st["scene"].refit(st["moved"], area_ref=st["area"])
        H = et.simulate(ctx, st["scene"], st["sim"], paths=st["paths"], ws=st["ws"], out=st["out"])
        P = st["paths"]
        res = {"H": H, "count": P.count}
        if kind == "frame":
            res["curvature"], res["vertex_curvature"] = st["scene"].curvature()
        if st["keep"]:
            res.update(p=P.p, rtot=P.rtot, dout=P.dout, tri=P.tri, mat=P.mat, ray=P.ray, bounce=P.bounce, flags=P.flags)
        return res
    if kind == "batch":
        b = st["batch"]
        H = b.run(grad_spectra=st["grad"])
        # the parameters are float32, and so are the gradients that an optimiser takes
        return {"H": H} if st["grad"] is None else {"H": H, "grad_k": b.grad_k.float(), "grad_rx": b.grad_rx.float()}
    if kind == "synth":
        return et.synthesize(ctx, st["sim"], st["paths"], ws=st["ws"], out=st["out"])
    if kind == "fit":
        H = et.SpectraFn.apply(st["k"], st["place"] + st["shift"].double(), ctx, st["sim"], st["paths"])
        loss = torch.view_as_real(H - st["target"]).square().sum()
        gk, gx = torch.autograd.grad(loss, (st["k"], st["shift"]))
        return {"H": H.detach(), "grad_k": gk, "grad_shift": gx}
    if kind == "build":
        sc = et.Scene(ctx, st["mesh"], area_ref=st["area"])
        C, G = sc.curvature()
        i = sc.info()
        return {"curvature": C, "vertex_curvature": G, "nodes": int(i.n_nodes), "depth": int(i.depth), "cost": float(i.sah_cost)}
    h, dt = et.impulse_response(ctx, st["sim"], st["H"], st["n_t"], ws=st["ws"])
    return {"h": h, "signal": et.receiver_signal(ctx, h, st["call"], dt, ws=st["ws2"])}


def _triangles(case):
    if case["scene"] == "wall":
        return 2 + 32 * 19 * 2 + 64
    if case["scene"] == "foliage":
        return 16 * case["objects"]
    return 12 + case["objects"] // 2 * 972 + (case["objects"] - case["objects"] // 2) * 960


def work(case):
    """Bytes read and written once, and the flops of the plain sums (8 per record, receiver and bin for
    a spectrum, 16 for its adjoint).  Records of a traced pose: the share of rays that still hit at each
    bounce and the share in line of sight, as measured on these scenes."""
    kind = case["kind"]
    rec = 24 + 12 + 8 + 4 + 4 + 4 + 2
    if kind in ("pose", "frame", "batch"):
        jobs, tri = (case["jobs"], 12 + 350 * case["objects"]) if kind == "batch" else (1, _triangles(case))
        scene = case.get("scene", "room")
        hits = {"wall": 0.92, "room": float(case["bounces"]), "foliage": 0.81 * case["bounces"]}[scene] * case["rays"]
        seen = {"wall": 1.0, "room": 0.77, "foliage": 0.45}[scene]
        n = jobs * (hits + case.get("diff", 0) * (0.02 * case["objects"] if case.get("per_mesh") else 0.02))
        flops = 8.0 * n * seen * case["mics"] * case["bins"]
        b = 12 * jobs * case["rays"] + n * rec + 8.0 * jobs * case["mics"] * case["bins"] + 112.0 * tri
        if case.get("adjoint"):
            flops, b = 3 * flops, b + 8.0 * jobs * case["mics"] * case["bins"]
        if kind == "frame":
            b += 200.0 * tri
        return {"bytes": b, "flops": flops}
    if kind in ("synth", "fit"):
        terms = 0.7 * case["records"] * case["mics"] * case["bins"]
        H = 8.0 * case["mics"] * case["bins"]
        return {"bytes": case["records"] * rec + (H if kind == "synth" else 3 * H), "flops": terms * (8 if kind == "synth" else 24)}
    if kind == "build":
        # mesh in (20 B a triangle, 6 B of vertices), nodes, triangles, curvature and lists out
        return {"bytes": _triangles(case) * (26.0 + 64 + 48 + 8 + 8 + 4 + 12), "flops": 1000.0 * _triangles(case)}
    M, n, L = case["mics"], case["samples"], case["call"]
    return {"bytes": 8.0 * M * case["bins"] + 4.0 * M * n + 4.0 * L + 4.0 * M * (n + L - 1),
            "flops": 5.0 * M * n * math.log2(n) * 4}


# ------------------------------------------------------------------ 64-bit values

def _spectra(case, seed):
    """Spectra of a few hundred echoes and a chirp, for the time domain."""
    g = np.random.default_rng(seed)
    M, F = case["mics"], case["bins"]
    f = np.linspace(20e3, 100e3, F)
    df = f[1] - f[0]
    tau = g.uniform(0, 0.9 / df, (M, 40))
    amp = g.exponential(1.0, (M, 40)) * np.exp(-3 * tau * df)
    H = np.zeros((M, F), complex)
    for e in range(40):
        H += amp[:, e, None] * np.exp(2j * np.pi * np.mod(tau[:, e, None] * f, 1.0))
    dt = 1.0 / (case["samples"] * df)
    t = np.arange(case["call"]) * dt
    call = np.hanning(case["call"]) * np.sin(2 * math.pi * (20e3 * t + 40e3 * t * t / max(t[-1], dt)))
    sim = _settings(dict(case, bands=1), g, np.array(SENSOR), np.zeros((1, 3), np.float32), 1)
    return H.astype(np.complex64), call.astype(np.float32), sim


def _rows(F, Bk, Bd):
    """Runs of at most 64 bins within one material and one directivity band: first bin, length, bands."""
    k = np.arange(F, dtype=np.int64)
    b, d = k * Bk // F, k * max(Bd, 1) // F
    cut = np.flatnonzero(np.r_[True, (b[1:] != b[:-1]) | (d[1:] != d[:-1])])
    out = []
    for lo, hi in zip(cut, np.r_[cut[1:], F]):
        out += [(s, min(64, hi - s), b[lo], d[lo]) for s in range(lo, hi, 64)]
    return np.array(out)


def _gain(tab, v):
    """Bilinear gain of the cell-centred tables [Bd][El][Az] in directions v [n][3]: [n][Bd]."""
    Bd, El, Az = tab.shape
    fa = (torch.atan2(v[:, 1], v[:, 0]) + math.pi) / (2 * math.pi) * Az - 0.5
    fe = (torch.atan2(v[:, 2], torch.hypot(v[:, 0], v[:, 1])) + math.pi / 2) / math.pi * El - 0.5
    fe = torch.clamp(fe, 0.0, El - 1.0)
    i, j = torch.floor(fa), torch.floor(fe)
    ta, te = fa - i, fe - j
    i0, j0 = i.long() % Az, j.long()
    i1, j1 = (i0 + 1) % Az, torch.clamp(j0 + 1, max=El - 1)
    a0 = (1 - ta) * tab[:, j0, i0] + ta * tab[:, j0, i1]
    a1 = (1 - ta) * tab[:, j1, i0] + ta * tab[:, j1, i1]
    return ((1 - te) * a0 + te * a1).T


def _spectrum64(rec, s, m, k, x, dev):
    """Receiver m's spectrum in 64 bits: rows of at most 64 bins as products over the records."""
    F, (Q, Bk) = s["F"], s["refl_k"].shape
    tab = s.get("directivity")
    rows = _rows(F, Bk, 0 if tab is None else tab.shape[1])
    start = torch.as_tensor(rows[:, 0], dtype=torch.float64, device=dev)
    band, dband = (torch.as_tensor(rows[:, c], device=dev) for c in (2, 3))
    t64 = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=dev)  # noqa: E731
    beta, dc = t64(s["lobe_beta"]), t64(s["diff_coef"])
    df = (s["f_hi"] - s["f_lo"]) / (F - 1)
    w = x - rec["p"]
    leg = torch.linalg.norm(w, dim=1)
    u = w / leg[:, None]
    r = rec["rtot"] + leg
    d = rec["dout"]
    sin2 = torch.linalg.cross(d, u).square().sum(1)
    gam = torch.atan2(torch.sqrt(torch.where(sin2 > 0, sin2, torch.ones_like(sin2))) * (sin2 > 0), (d * u).sum(1))
    spec = k[rec["mat"]] * torch.exp(-gam[:, None] ** 2 / (2 * beta[rec["mat"]] ** 2))
    I = torch.where(rec["kind"][:, None] == 0, spec, dc[rec["mat"]])[:, band]
    if tab is not None:
        I = I * _gain(t64(tab[m]), -u)[:, dband]
    loss = -(s["atm_a0"] + s["atm_a1"] * s["f_lo"]) / 20 * math.log(10) * r - s["spreading_p"] * torch.log(r)
    slope = -s["atm_a1"] * df / 20 * math.log(10) * r
    c0, cb = r * (s["f_lo"] / s["c"]), r * (df / s["c"])
    cyc = c0[:, None] + start * cb[:, None]
    X = torch.polar(I * torch.exp(loss[:, None] + slope[:, None] * start), 2 * math.pi * (cyc - torch.floor(cyc.detach())))
    k2 = torch.arange(64, dtype=torch.float64, device=dev)
    Y = torch.polar(torch.exp(slope[:, None] * k2), 2 * math.pi * (k2 * cb[:, None]))
    blocks = X.transpose(0, 1).contiguous() @ Y
    at = torch.as_tensor(np.concatenate([i * 64 + np.arange(n) for i, n in enumerate(rows[:, 1])]), device=dev)
    return blocks.reshape(-1)[at]


def _exact_records(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    rec, s = _records(case, seed)
    seen = np.flatnonzero(rec["vis"])
    rec = {a: torch.as_tensor(b[seen]).to(dev) for a, b in rec.items()}
    rec["dout"], rec["mat"] = rec["dout"].double(), rec["mat"].long()
    n, step = len(seen), 20000
    parts = [{a: b[i:i + step] for a, b in rec.items()} for i in range(0, n, step)]
    k = torch.as_tensor(s["refl_k"]).double().to(dev)
    x = torch.as_tensor(s["rx_pos"]).to(dev)
    with torch.no_grad():
        H = torch.stack([sum(_spectrum64(p, s, m, k, x[m], dev) for p in parts) for m in range(case["mics"])])
    if case["kind"] == "synth":
        return H.cpu()
    g = 2 * (H - torch.as_tensor(_target(case, seed)).to(dev))
    k.requires_grad_(True)
    x.requires_grad_(True)
    gk, gx = torch.zeros_like(k), torch.zeros_like(x)
    for m in range(case["mics"]):
        for p in parts:
            a, b = torch.autograd.grad(_spectrum64(p, s, m, k, x[m], dev), (k, x), g[m])
            gk, gx = gk + a, gx + b
    return {"H": H.cpu(), "grad_k": gk.cpu(), "grad_shift": gx.cpu()}


def _exact_curvature(mesh, area_ref):
    """Cotangent-operator curvature per vertex and its weighted spread per triangle."""
    V, t = mesh["vertices"].astype(np.float64), mesh["tris"].astype(np.int64)
    P = V[t]
    area2 = np.linalg.norm(np.cross(P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]), axis=1)
    ok = 0.5 * area2 >= 1e-20
    dot = np.stack([((P[:, (c + 1) % 3] - P[:, c]) * (P[:, (c + 2) % 3] - P[:, c])).sum(1) for c in range(3)], 1)
    cot = dot / np.where(ok, area2, 1.0)[:, None]
    obtuse = (dot < 0).any(1)
    K, A = np.zeros_like(V), np.zeros(len(V))
    for c in range(3):
        c1, c2 = (c + 1) % 3, (c + 2) % 3
        ea, eb = P[:, c] - P[:, c1], P[:, c] - P[:, c2]
        voronoi = ((ea * ea).sum(1) * cot[:, c2] + (eb * eb).sum(1) * cot[:, c1]) / 8
        mixed = np.where(~obtuse, voronoi, 0.5 * area2 * np.where(dot[:, c] < 0, 0.5, 0.25))
        np.add.at(K, t[ok, c], (cot[:, c2, None] * ea + cot[:, c1, None] * eb)[ok])
        np.add.at(A, t[ok, c], mixed[ok])
    G = np.where(A > 0, np.linalg.norm(K, axis=1) / (4 * np.where(A > 0, A, 1.0)), 0.0)
    spread = G[t].max(1) - G[t].min(1)
    return np.minimum(1.0, 0.5 * area2 / area_ref) * spread, G


def exact(case, seed):
    kind = case["kind"]
    if kind in ("synth", "fit"):
        return _exact_records(case, seed)
    if kind == "build":
        mesh = _mesh(case, np.random.default_rng(seed))
        C, G = _exact_curvature(mesh, _area_ref(mesh))
        return {"curvature": C, "vertex_curvature": G, "nodes": None, "depth": None, "cost": None}
    if kind == "signal":
        H, call, _ = _spectra(case, seed)
        n_t, f_lo, df = case["samples"], 20e3, 80e3 / (case["bins"] - 1)
        n = np.arange(n_t)
        dt = 1.0 / (n_t * df)
        cyc = np.mod(f_lo * dt * n, 1.0)
        h = 2 * df * (np.exp(-2j * np.pi * cyc) * np.fft.fft(H.astype(np.complex128), n_t, axis=1)).real
        size = n_t + case["call"] - 1
        s = dt * np.fft.irfft(np.fft.rfft(h, 2 * size) * np.fft.rfft(call.astype(np.float64), 2 * size), 2 * size)[:, :size]
        return {"h": h, "signal": s}
    return None
