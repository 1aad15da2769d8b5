"""Sizes at the edges of the kernels' splits, against the FP64 oracle: rays per wave and triangles per tree of the
traversal (partly filled waves, empty node slots, jobs that share a wave), mesh sizes around the
sort's and the scan's blocks, band layouts whose rows are cut off 64-bin boundaries, and lengths around the transforms'
splits."""

import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_parity import check_spectra, compare_traces

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(et):
    return et.Context(0)


def _soup(T, seed):
    """T random triangles (30-100 cm) in a 4 m box ahead of the emitter."""
    g = W.rng(seed)
    c = g.uniform([1.0, -2.0, -2.0], [5.0, 2.0, 2.0], (T, 3))
    v = (c[:, None, :] + g.normal(0, 0.4, (T, 3, 3))).reshape(-1, 3).astype(np.float32)
    return {"vertices": v, "tris": np.arange(3 * T, dtype=np.int32).reshape(T, 3), "tri_material": np.zeros(T, np.int32),
            "tri_object": np.zeros(T, np.int32), "n_objects": 1}


@pytest.mark.parametrize("T,N", [(3, 1), (4, 15), (5, 16), (6, 17), (9, 63), (40, 65), (1000, 130), (1000, 20011),
                                 (2048, 333), (2049, 333), (8193, 333)])
def test_traces_of_random_triangles(et, ctx, T, N):
    """Every certified ray's hits, shadow rays included, as the oracle's brute force finds them; per-receiver line of
    sight too."""
    scene = _soup(T, 100 + T)
    _, sim = W.tiny_scene(n_rays=N)
    sc = et.Scene(ctx, scene)
    ref = O.trace(scene, sim)
    gpu = et.trace(ctx, sc, et.Sim(sim)).to_host()
    assert compare_traces(gpu, ref, ref["certified"]) == 0
    per = dict(sim, per_rx_visibility=True)
    ref = O.trace(scene, per)
    dirs = sim["ray_dirs"][ref["certified"]]
    if len(dirs):
        ref = O.trace(scene, per, dirs=dirs)
        h = et.trace(ctx, sc, et.Sim(per, ray_dirs=dirs)).to_host()
        key = {(int(r), int(b)): int(x) for r, b, x in zip(ref["ray"], ref["bounce"], ref["rxvis"])}
        assert {(int(r), int(b)): int(x) for r, b, x in zip(h["ray"], h["bounce"], h["rxvis"])} == key


@pytest.mark.parametrize("rays", [(1, 3, 5), (10, 37, 70), (64, 1, 200)])
def test_batch_jobs_that_share_waves(et, ctx, rays):
    """Jobs of fewer rays than a wave holds, over scenes of their own (one without triangles): each job's spectra
    against its own oracle trace.  Spectra within the factorised kernel's 1e-4."""
    scenes = [_soup(300, 7), _soup(5, 8), {**_soup(1, 9), "tris": np.zeros((0, 3), np.int32),
                                            "tri_material": np.zeros(0, np.int32), "tri_object": np.zeros(0, np.int32)}]
    sims, refs = [], []
    for i, n in enumerate(rays):
        _, sim = W.tiny_scene(seed=50 + i, n_rays=4 * n + 16, F=256)
        cert = O.trace(scenes[i], sim)["certified"]
        # (lobes wide enough that no reflection's factor leaves FP32's range)
        sim = dict(sim, ray_dirs=sim["ray_dirs"][cert][:n], lobe_beta=np.full_like(sim["lobe_beta"], 1.0))
        refs.append(O.synth(O.trace(scenes[i], sim), sim))
        sims.append(et.Sim(sim, flags=et.ET_SPECULAR))
    H = et.Batch(ctx, [(et.Scene(ctx, sc), s) for sc, s in zip(scenes, sims)]).run().cpu().numpy()
    for i in range(len(rays)):
        if np.any(refs[i]):
            check_spectra(H[i], refs[i], f"job {i} of {rays[i]} rays")
        else:
            assert not np.any(H[i])


@pytest.mark.parametrize("F,Bk,Q,mics,table", [(31, 1, 1, 1, False), (97, 3, 2, 2, False), (200, 7, 3, 5, True),
                                               (1000, 16, 16, 3, False), (2049, 5, 2, 33, False), (2080, 13, 4, 2, True),
                                               (4100, 33, 2, 1, True)])
def test_rows_off_the_64_bin_blocks(et, ctx, F, Bk, Q, mics, table):
    """Bands that end inside a 64-bin block (with a directivity's own bands beside the material's), part rows at the
    end of the grid, receivers that do not fill a group."""
    scene, sim = W.tiny_scene(n_rays=3000)
    g = W.rng(F + Bk)
    scene = dict(scene, tri_material=g.integers(0, Q, len(scene["tris"])).astype(np.int32))
    sim = dict(sim, F=F, refl_k=g.uniform(0.3, 0.99, (Q, Bk)).astype(np.float32),
               lobe_beta=g.uniform(0.05, 0.3, (Q, Bk)).astype(np.float32),
               diff_coef=g.uniform(0.05, 0.3, (Q, Bk)).astype(np.float32),
               rx_pos=np.asarray(sim["rx_pos"])[:1] + g.normal(0, 0.02, (mics, 3)),
               rx_rot=np.stack([W.frame_from_forward(v) for v in g.normal(size=(mics, 3))]))
    if table:
        sim["directivity"] = W.directivity_table(g, mics, Bd=6, El=8, Az=16)
    ref = O.trace(scene, sim, certify=False)
    H = et.synthesize(ctx, et.Sim(sim), et.Paths.from_records(ref)).cpu().numpy()
    check_spectra(H, O.synth(ref, sim), f"F={F}, {Bk} bands: kernel {ctx.stats().synth_kernel}")


@pytest.mark.parametrize("sigma", [1, -1])
@pytest.mark.parametrize("F,n_t", [(2, 2), (3, 4), (5, 8), (16, 16), (20, 32), (33, 64), (100, 128), (256, 256),
                                   (300, 512), (1000, 1024), (700, 2048), (4096, 4096), (5000, 8192), (9000, 16384),
                                   (4097, 32768), (32768, 32768), (500, 65536)])
def test_impulse_response_lengths(et, ctx, F, n_t, sigma):
    """Every transform length, with the bins ending inside and past the first residue's points, against FP64.  Up to 16
    levels of additions and five products, rounded to 6e-8 of the value each and independently, stay
    below 1e-6 of the norm."""
    import torch
    g = W.rng(F)
    _, sim = W.tiny_scene(n_rays=16)
    M = 3
    sim = dict(sim, F=F, phase_sign=sigma, rx_pos=np.zeros((M, 3)), rx_rot=np.stack([np.eye(3)] * M))
    H = (g.normal(size=(M, F)) + 1j * g.normal(size=(M, F))).astype(np.complex64)
    h, dt = et.impulse_response(ctx, et.Sim(sim), torch.as_tensor(H).cuda(), n_t)
    df = (sim["f_hi"] - sim["f_lo"]) / (F - 1)
    X = np.zeros((M, n_t), complex)
    X[:, :F] = H
    S = np.fft.fft(X, axis=1) if sigma > 0 else np.fft.ifft(X, axis=1) * n_t
    cyc = sim["f_lo"] * np.arange(n_t) / (n_t * df)
    ref = 2 * df * np.real(np.exp(-2j * np.pi * sigma * (cyc - np.floor(cyc))) * S)
    e = np.linalg.norm(h.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"F={F}, {n_t} samples: {e:.2e}")
    assert e <= 1e-6


@pytest.mark.parametrize("n_t,L", [(1, 1), (1, 40), (64, 1), (512, 2), (1024, 512), (1024, 513), (4096, 1024), (4096, 1025),
                                   (2048, 2049), (16384, 640), (512, 4096), (8192, 4097)])
def test_convolution_lengths(et, ctx, n_t, L):
    """Blocks of every length, the last one part filled, responses shorter than the call; against FP64, 1e-6 of the norm
    (three transforms of up to 14 levels, rounded independently)."""
    import torch
    g = W.rng(n_t + L)
    h = g.normal(size=(3, n_t)).astype(np.float32)
    call = g.normal(size=L).astype(np.float32)
    out = et.receiver_signal(ctx, torch.as_tensor(h).cuda(), torch.as_tensor(call).cuda(), 2e-6).cpu().numpy()
    n = n_t + L - 1
    ref = 2e-6 * np.fft.ifft(np.fft.fft(h.astype(float), n, axis=1) * np.fft.fft(call.astype(float), n), axis=1).real
    e = np.linalg.norm(out - ref) / np.linalg.norm(ref)
    print(f"{n_t} samples, call of {L}: {e:.2e}")
    assert out.shape == (3, n) and e <= 1e-6


@pytest.mark.parametrize("rim,extra", [(3, 0), (8, 0), (9, 1), (64, 0), (65, 2), (200, 1)])
def test_curvature_of_fans(et, ctx, rim, extra):
    """A vertex of 8, 9, 64, 65 and 200 triangles (eight lanes or a wave per vertex), triangles that repeat a vertex and
    without area among them: bit for bit the oracle's sums in triangle order."""
    g = W.rng(rim)
    ang = np.linspace(0, 2 * np.pi, rim, endpoint=False)
    v = [[3.0, 0.0, 0.3]] + [[3.0 + g.normal(0, 0.05), np.cos(a), np.sin(a)] for a in ang]
    t = [[0, 1 + i, 1 + (i + 1) % rim] for i in range(rim)]
    for k in range(extra):
        t.insert(2 + 3 * k, [0, 0, 1 + k])
    n = len(t)
    scene = {"vertices": np.asarray(v, np.float32), "tris": np.asarray(t, np.int32), "tri_material": np.zeros(n, np.int32),
             "tri_object": (np.arange(n) * 70 // n).astype(np.int32), "n_objects": 70}
    C, G = et.Scene(ctx, scene, area_ref=0.01).curvature()
    G_ref, C_ref = O.curvature(scene, 0.01)
    assert np.array_equal(C.cpu().numpy(), C_ref) and np.array_equal(G.cpu().numpy(), G_ref)


@pytest.mark.parametrize("T", [2, 3, 224, 225, 2047, 2049, 6000])
def test_refit_equals_build(et, ctx, T):
    """Mesh sizes around the clustering's workgroups and tail and the refit's narrow levels: a scene refitted to moved
    vertices hits what a scene built on them hits."""
    a, b = _soup(T, 300 + T), _soup(T, 300 + T)
    b["vertices"] = (a["vertices"] + W.rng(T).normal(0, 0.05, a["vertices"].shape)).astype(np.float32)
    _, sim = W.tiny_scene(n_rays=2000)
    s = et.Sim(sim)
    moved, built = et.Scene(ctx, a), et.Scene(ctx, b)
    assert moved.info().n_nodes == T - 1 and built.info().depth <= 64
    moved.refit(b["vertices"])
    x, y = et.trace(ctx, moved, s).to_host(), et.trace(ctx, built, s).to_host()
    for k in ("ray", "bounce", "tri", "vis"):
        assert np.array_equal(x[k], y[k]), k


@pytest.mark.parametrize("per_mesh,per_rx", [(False, False), (True, False), (True, True)])
def test_diffraction_beside_the_walks(et, ctx, per_mesh, per_rx):
    """Rays and samples in one call (drawn beside the walks) give the rays' records and then the samples' records of the
    two calls apart (which run in order), call after call, and the same number of shadow rays; also with
    the call on a stream of its own and captured in a graph (in order there), replayed between eager calls."""
    import torch
    scene = W.room_geometry(W.rng(31), n_boxes=8, n_cyl=8)
    _, base = W.room_scene(n_rays=1 << 14, M=3, F=256, diff_K=64 if per_mesh else 3000)
    flag = (et.ET_DIFF_PER_MESH if per_mesh else 0) | (et.ET_PER_RX_VISIBILITY if per_rx else 0)
    sim = dict(base, diff_max_meshes=scene["n_objects"], emitter_pos=[1.0, 4.0, 1.2])
    sc = et.Scene(ctx, scene, area_ref=W.median_triangle_area(scene))
    both = et.Sim(sim, flags=et.ET_SPECULAR | et.ET_DIFFRACTION | flag)
    keys = ("ray", "bounce", "tri", "vis", "rtot", "p", "rxvis")
    parts, shadow = [], 0
    for f in (et.ET_SPECULAR, et.ET_DIFFRACTION):
        parts.append(et.trace(ctx, sc, et.Sim(sim, flags=f | flag)).to_host())
        shadow += ctx.stats().shadow_rays
    ref = {k: np.concatenate([x[k] for x in parts]) for k in keys}
    assert len(parts[0]["ray"]) and len(parts[1]["ray"])

    def check(P):
        h = P.to_host()
        for k in keys:
            assert np.array_equal(h[k], ref[k]), k

    for _ in range(5):
        check(et.trace(ctx, sc, both))
        assert ctx.stats().shadow_rays == shadow
    P, ws = et.Paths(both.capacity()), et.Workspace()
    out = torch.empty(3, 256, 2, device="cuda")
    H = et.simulate(ctx, sc, both, paths=P, ws=ws, out=out).clone()
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        et.simulate(ctx, sc, both, paths=P, ws=ws, out=out)
        check(P)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            et.simulate(ctx, sc, both, paths=P, ws=ws, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_complex(out), H)
        assert torch.equal(et.simulate(ctx, sc, both), H)
        torch.cuda.synchronize()


@pytest.mark.parametrize("seed", range(10))
def test_any_band_layout_matches_the_per_term_kernel(et, ctx, seed):
    """Random grids, band counts, directivities and readings (direct paths, path product, per-receiver visibility): the
    kernel the layout takes against the per-term one on the same records.  Both are within 4e-6 of the FP64 sum."""
    g = W.rng(700 + seed)
    F, Bk, Q, M = int(np.exp(g.uniform(np.log(2), np.log(5000)))), int(g.integers(1, 18)), int(g.integers(1, 6)), int(g.integers(1, 7))
    scene = _soup(200, 40 + seed)
    scene["tri_material"] = g.integers(0, Q, 200).astype(np.int32)
    _, sim = W.tiny_scene(n_rays=4000)
    sim = dict(sim, F=F, refl_k=g.uniform(0.3, 0.99, (Q, Bk)).astype(np.float32),
               lobe_beta=g.uniform(0.3, 1.0, (Q, Bk)).astype(np.float32),
               diff_coef=g.uniform(0.05, 0.3, (Q, Bk)).astype(np.float32),
               rx_pos=g.normal(0, 0.05, (M, 3)), rx_rot=np.stack([W.frame_from_forward(v) for v in g.normal(size=(M, 3))]))
    if seed % 2:
        sim["directivity"] = W.directivity_table(g, M, Bd=int(g.integers(1, 9)), El=8, Az=16)
    if seed % 3 == 1:
        sim["passive_coef"] = g.uniform(0.2, 1.0, Bk).astype(np.float32)
    flags = et.ET_SPECULAR | (et.ET_PASSIVE if sim.get("passive_coef") is not None else 0)
    flags |= et.ET_PATH_PRODUCT if seed % 5 == 2 else 0
    flags |= et.ET_PER_RX_VISIBILITY if seed % 4 == 3 else 0
    s = et.Sim(sim, flags=flags)
    P = et.trace(ctx, et.Scene(ctx, scene), s)
    H = et.synthesize(ctx, s, P).cpu().numpy()
    k = ctx.stats().synth_kernel
    D = et.synthesize(ctx, et.Sim(sim, flags=flags | et.ET_SYNTH_DIRECT), P).cpu().numpy()
    check_spectra(H, D, f"F={F}, {Bk} bands, {M} receivers, flags {flags}: kernel {k}", tol=1e-5)


@pytest.mark.parametrize("F,jobs,kernel,rows", [(256, "hh", 1, 0), (256, "hr", 2, 1), (256, "rh", 2, 1), (250, "hh", 2, 1), (250, "hrr", 2, 1),
                                                (256, "ht", 2, 0), (250, "rt", 2, 0), (2100, "rrr", 2, 1)])
def test_batch_takes_one_kernel_for_its_jobs(et, ctx, F, jobs, kernel, rows):
    """Jobs whose own layouts call for halves (bands on whole runs of 64 bins), rows (a directivity of three bands) and single
    terms (asked for): the batch runs them all by the most general one, each job as it comes out alone.
    The kernel in halves is within 2e-6 of the sum on such spectra, those in FP32 within 1e-6; 4e-6 between two."""
    g = W.rng(F)
    scenes = [et.Scene(ctx, _soup(120, 60 + i)) for i in range(2)]
    sims = []
    for i, k in enumerate(jobs):
        _, sim = W.tiny_scene(seed=70 + i, n_rays=900 + 100 * i, F=F)
        sim = dict(sim, refl_k=g.uniform(0.3, 0.99, (1, 4)).astype(np.float32), lobe_beta=np.full((1, 4), 1.0, np.float32),
                   diff_coef=np.full((1, 4), 0.1, np.float32))
        if k == "r":
            sim["directivity"] = W.directivity_table(g, len(sim["rx_pos"]), Bd=3, El=8, Az=16)
        sims.append(et.Sim(sim, flags=et.ET_SPECULAR | (et.ET_SYNTH_DIRECT if k == "t" else 0)))
    b = et.Batch(ctx, [(scenes[i % 2], s) for i, s in enumerate(sims)])
    H = b.run().cpu().numpy()
    st = ctx.stats()
    assert (st.synth_kernel, st.synth_rows) == (kernel, rows)
    for i, s in enumerate(sims):
        check_spectra(H[i], et.simulate(ctx, scenes[i % 2], s).cpu().numpy(), f"{F} bins, job {i} of {jobs}", tol=4e-6)
