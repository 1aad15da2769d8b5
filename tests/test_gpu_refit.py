"""Dynamic scenes: a BVH refit over new vertex positions (et_scene_refit) against a fresh
build of the moved scene and against the FP64 oracle.

  * refitting to the build's own vertices reproduces the scene blob bit for bit (boxes are
    exact unions of FP32 triangle bounds, curvature is recomputed in the same order);
  * after an animation frame (objects turned, moved, some deformed) the refitted scene gives
    bit-identical curvature and trace records to a fresh build of the moved scene, and the
    oracle's hits on certified rays;
  * refitting back to the first frame restores the first blob bit for bit.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(et):
    return et.Context(0)


@pytest.fixture(scope="module")
def frames():
    scene, sim = W.room_scene(n_rays=1 << 18, diff_K=16384)
    V1 = W.animate_objects(scene, W.rng(31))
    moved = dict(scene, vertices=V1)
    return scene, moved, sim


def _records(P):
    h = P.to_host()
    h.pop("count")
    order = np.lexsort((h["bounce"], h["ray"]))
    return {k: np.asarray(v)[order] for k, v in h.items()}


def test_refit_same_vertices_reproduces_build(et, ctx, frames):
    scene, _, sim = frames
    sc = et.Scene(ctx, scene, area_ref=sim["area_ref"])
    blob0 = sc.blob.clone()
    sc.refit(scene["vertices"], area_ref=sim["area_ref"])
    info = sc.info()
    print(f"room: build {info.build_ms:.2f} ms, refit {info.refit_ms:.2f} ms, T {info.T}")
    assert info.refit_ms > 0
    assert torch_equal(sc.blob, blob0)


def torch_equal(a, b):
    import torch
    return bool(torch.equal(a, b))


def test_refit_frame_matches_fresh_build_and_oracle(et, ctx, frames):
    scene, moved, sim = frames
    a_ref = sim["area_ref"]
    sc = et.Scene(ctx, scene, area_ref=a_ref)
    blob0 = sc.blob.clone()
    sah0 = sc.info().sah_cost
    sc.refit(moved["vertices"], area_ref=a_ref)
    fresh = et.Scene(ctx, moved, area_ref=a_ref)
    ri, fi = sc.info(), fresh.info()
    print(f"moved room: SAH refit {ri.sah_cost:.1f} (first frame {sah0:.1f}), fresh build {fi.sah_cost:.1f}; "
          f"refit {ri.refit_ms:.2f} ms vs build {fi.build_ms:.2f} ms")
    assert ri.sah_cost >= 0.95 * fi.sah_cost   # a refit never beats a fresh build by much

    # curvature: bit-identical to the fresh build and to the oracle (Eq. 1)
    C1, G1 = sc.curvature()
    C2, G2 = fresh.curvature()
    assert torch_equal(C1, C2) and torch_equal(G1, G2)
    G_ref, C_ref = O.curvature(moved, a_ref)
    assert np.array_equal(C1.cpu().numpy(), C_ref) and np.array_equal(G1.cpu().numpy(), G_ref)

    # specular trace over all rays: identical records, triangles included.  Closest-hit ties go
    # to the smaller triangle index and box culling is widened beyond rounding, so the hit does
    # not depend on the tree's topology.
    s = et.Sim(sim, flags=et.ET_SPECULAR)
    ra = _records(et.trace(ctx, sc, s))
    assert ctx.stats().stack_overflows == 0
    rb = _records(et.trace(ctx, fresh, s))
    assert ra.keys() == rb.keys()
    for k in ra:
        if k != "tri":
            assert np.array_equal(ra[k], rb[k]), k
    diff = np.nonzero(ra["tri"] != rb["tri"])[0]
    print(f"moved room: {len(ra['ray'])} records, {len(diff)} with another (tied) triangle")
    assert len(diff) == 0

    # the oracle on a seeded subset of rays of the moved scene
    sub = np.sort(W.rng(32).choice(len(sim["ray_dirs"]), 1024, replace=False))
    dirs = sim["ray_dirs"][sub]
    ref = O.trace(moved, sim, dirs=dirs)
    gpu = et.trace(ctx, sc, et.Sim(sim, flags=et.ET_SPECULAR, ray_dirs=dirs)).to_host()
    from test_gpu_parity import compare_traces
    mism = compare_traces(gpu, ref, ref["certified"])
    print(f"moved room subset: certified {ref['certified'].mean():.4f}, mismatches {mism}")
    assert mism == 0

    # full simulation with diffraction (curvature-driven sampling) matches the fresh build
    full = et.Sim(sim)
    Ha = et.simulate(ctx, sc, full).cpu().numpy()
    Hb = et.simulate(ctx, fresh, full).cpu().numpy()
    assert np.array_equal(Ha, Hb)

    # back to the first frame
    sc.refit(scene["vertices"], area_ref=a_ref)
    assert torch_equal(sc.blob, blob0)


def test_refit_rejects_bad_arguments(et, ctx, frames):
    import ctypes
    scene, _, sim = frames
    sc = et.Scene(ctx, scene)
    with pytest.raises(ValueError):
        sc.refit(scene["vertices"][:-1])
    v = ctypes.c_void_p(sc.vertices.data_ptr())
    assert et.lib().et_scene_refit(ctx.h, sc.h, None, 0.0) == -1          # no vertices
    assert et.lib().et_scene_refit(ctx.h, None, v, 0.0) == -1             # no scene
    assert et.lib().et_scene_refit(ctx.h, sc.h, v, float("nan")) == -1    # area_ref not finite


def test_half_a_billion_vertices(et):
    """2^29 + 40 vertices, nearly all of them in no triangle (a launch with eight threads per vertex would take more than
    2^32 of them): the curvature of a fan over the last ones, built and refitted, is the small mesh's."""
    import torch
    ctx = et.Context(0)
    V, rim = (1 << 29) + 40, 39
    ang = np.linspace(0, 2 * np.pi, rim, endpoint=False)
    fan = np.concatenate([[[3.0, 0.0, 0.3]], np.stack([3.0 + 0.05 * np.sin(3 * ang), np.cos(ang), np.sin(ang)], 1)]).astype(np.float32)
    t = np.array([[0, 1 + i, 1 + (i + 1) % rim] for i in range(rim)], np.int32)
    rest = {"tri_material": np.zeros(rim, np.int32), "tri_object": np.zeros(rim, np.int32), "n_objects": 1}
    small = et.Scene(ctx, {"vertices": fan, "tris": t, **rest}, area_ref=0.01)
    v = torch.zeros(V, 3, device="cuda")
    v[-40:] = torch.as_tensor(fan, device="cuda")
    large = et.Scene(ctx, {"vertices": v, "tris": t + np.int32(V - 40), **rest}, area_ref=0.01)
    for scale in (1.0, 1.25):
        if scale != 1.0:
            small.refit(fan * np.float32(scale), area_ref=0.01)
            large.refit(v * scale, area_ref=0.01)
        (C, G), (C1, G1) = small.curvature(), large.curvature()
        assert torch.equal(C, C1) and torch.equal(G, G1[-40:]) and float(G.min()) > 0
        assert int(torch.count_nonzero(G1)) == 40
