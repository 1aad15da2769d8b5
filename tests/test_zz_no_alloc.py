"""et_synthesize_noalloc (no workspace: the library's per-device scratch, every record walked)
against et_synthesize on the same records, through the C ABI: two calls in a row, the first on
the room scene's records (32 receivers x 4096 bins), the second with a smaller input (the tiny
scene: 2 receivers x 1024 bins, fewer records), then the per-term kernel; each within the
1e-4 relative L2 bar, over all receivers and per receiver."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import check_spectra

pytestmark = pytest.mark.gpu


def _records(et, ctx, scene, sim, n_rays):
    sc = et.Scene(ctx, scene, area_ref=sim.get("area_ref", 0.0))
    s = et.Sim(sim, ray_dirs=sim["ray_dirs"][:n_rays])
    return s, et.trace(ctx, sc, s)


def test_noalloc_synthesis_matches_workspace_call(et):
    import torch
    ctx = et.Context(0)
    room, rsim = W.room_scene(n_rays=1 << 20)
    tiny, tsim = W.tiny_scene()
    s1, P1 = _records(et, ctx, room, rsim, 1 << 16)
    s2, P2 = _records(et, ctx, tiny, tsim, 4096)
    s3 = et.Sim(tsim, flags=et.ET_SPECULAR | et.ET_SYNTH_DIRECT, ray_dirs=tsim["ray_dirs"][:4096])
    cases = [("room, 32 x 4096", s1, P1), ("tiny, 2 x 1024 (smaller input)", s2, P2), ("tiny, per-term kernel", s3, P2)]
    outs = [torch.empty(s.M, s.F, 2, dtype=torch.float32, device="cuda") for _, s, _ in cases]
    torch.cuda.synchronize()
    for (what, s, P), out in zip(cases, outs):
        ref = et.synthesize(ctx, s, P).cpu().numpy()
        kref = ctx.stats().synth_kernel
        H = et.synthesize_noalloc(ctx, s, P, out).cpu().numpy()
        st = ctx.stats()
        print(f"{what}: {P.n()} records, kernel {st.synth_kernel}")
        assert st.synth_kernel == kref
        assert np.all(np.isfinite(H)) and np.linalg.norm(ref) > 0
        check_spectra(H, ref, f"allocation-free synthesis vs workspace call ({what})")
    # the scratch keeps the last call's contents: a repeated call still starts from zero
    H = et.synthesize_noalloc(ctx, s1, P1, outs[0]).cpu().numpy()
    check_spectra(H, et.synthesize(ctx, s1, P1).cpu().numpy(), "room again after smaller calls")


def test_noalloc_per_term_where_the_rows_do_not_fit(et):
    """Receivers and bins whose partial spectra fill the scratch but for 8 KB, bands off the 64-bin blocks: the row table does
    not fit beside them, so the call runs per term; the workspace call, over rows.  Sampled bins against the
    oracle: 4e-6 over rows; per term the phase's step per bin is rounded to 2^-33 cycles, 1e-4 of a turn's radius at
    the last of 131,056 bins."""
    import torch

    import oracle as O
    M, F, Bk = 64, 131056, 7
    g = W.rng(3)
    scene, sim = W.tiny_scene(n_rays=256)
    sim = dict(sim, F=F, rx_pos=g.normal(0, 0.05, (M, 3)), rx_rot=np.repeat(np.eye(3)[None], M, 0),
               refl_k=g.uniform(0.3, 0.99, (1, Bk)).astype(np.float32), lobe_beta=np.full((1, Bk), 1.0, np.float32),
               diff_coef=np.full((1, Bk), 0.1, np.float32))
    ref = O.trace(scene, sim, certify=False)
    ref = {k: (v[:40] if isinstance(v, np.ndarray) and len(v) == len(ref["rtot"]) else v) for k, v in ref.items()}
    ctx, s, P = et.Context(0), et.Sim(sim, flags=et.ET_SPECULAR), et.Paths.from_records(ref)
    H = et.synthesize(ctx, s, P)
    assert ctx.stats().synth_kernel == 2 and ctx.stats().synth_rows == 1
    N = et.synthesize_noalloc(ctx, s, P, torch.empty(M, F, 2, device="cuda"))
    assert ctx.stats().synth_kernel == 2 and ctx.stats().synth_rows == 0
    bins = np.sort(g.choice(F, 300, replace=False))
    want = O.synth(ref, sim, bins=bins)
    check_spectra(H.cpu().numpy()[:, bins], want, "over rows, sampled bins", tol=4e-6)
    check_spectra(N.cpu().numpy()[:, bins], want, "per term, sampled bins", tol=1e-4)
