"""Records with unusual contents, through every form of the forward synthesis: records that do not count (hidden ones, and
passive ones of another receiver) hold anything, and add nothing, in the allocation-free call too, which walks every record;
the lobe widths of a material belong to its specular records alone."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_parity import check_spectra

pytestmark = pytest.mark.gpu

# bins, material bands, directivity bands: edges on 512 and 256 bins, on 64, inside a row, a single bin, and (64 bands of
# 64 bins) the per-term kernel
LAYOUTS = [(1024, 2, 0), (1024, 4, 4), (960, 5, 0), (960, 5, 3), (200, 7, 0), (4100, 7, 5), (1, 1, 0), (4096, 64, 0)]


@pytest.fixture(scope="module")
def ctx(et):
    return et.Context(0)


def _sim(F, Bk, Bd, Q=3, M=3, seed=5):
    g = W.rng(seed + F + Bk)
    _, sim = W.tiny_scene(n_rays=1024)
    sim = dict(sim, F=F, refl_k=g.uniform(0.3, 0.99, (Q, Bk)).astype(np.float32),
               lobe_beta=g.uniform(0.3, 1.0, (Q, Bk)).astype(np.float32),
               diff_coef=g.uniform(0.05, 0.3, (Q, Bk)).astype(np.float32),
               passive_coef=g.uniform(0.2, 1.0, Bk).astype(np.float32),
               rx_pos=g.normal(0, 0.05, (M, 3)), rx_rot=np.stack([W.frame_from_forward(v) for v in g.normal(size=(M, 3))]))
    if F == 1:
        sim["f_hi"] = sim["f_lo"]
    if Bd:
        sim["directivity"] = W.directivity_table(g, M, Bd=Bd, El=8, Az=16)
    return sim, g


def _records(g, n, Q, M, kinds=(0, 0, 0, 1, 2)):
    kind = g.choice(kinds, n).astype(np.uint8)
    d = g.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    d[kind != 0] = 0
    mat = np.where(kind == 2, g.integers(0, M, n), g.integers(0, Q, n)).astype(np.int32)
    return dict(p=g.normal(0, 1, (n, 3)) + [3.0, 0, 0], dout=d.astype(np.float32), rtot=g.uniform(1, 6, n), mat=mat, kind=kind,
                vis=np.ones(n, np.uint8), tri=np.zeros(n, np.int32))


def _forms(et, ctx, sim, flags, P):
    import torch
    s = et.Sim(sim, flags=flags)
    yield "workspace", et.synthesize(ctx, s, P).cpu().numpy()
    out = torch.empty(s.M, s.F, 2, device="cuda")
    yield "allocation-free", et.synthesize_noalloc(ctx, s, P, out).cpu().numpy()


@pytest.mark.parametrize("direct", [False, True])
@pytest.mark.parametrize("hidden", ["nan", "inf", "receiver", "material"])
@pytest.mark.parametrize("layout", LAYOUTS)
def test_hidden_records_hold_anything(et, ctx, layout, hidden, direct):
    """Points and directions that are NaN or infinite, points on a receiver, and materials outside the tables, in records that
    are hidden, beside 300 that count; the oracle's spectra of those 300 (4e-6: FP32 terms)."""
    sim, g = _sim(*layout)
    M, Q = len(sim["rx_pos"]), 3
    rec = _records(g, 700, Q, M)
    off = np.ones(700, bool)
    off[g.choice(700, 300, replace=False)] = False
    rec["vis"][off] = 0
    if hidden in ("nan", "inf"):
        v = np.nan if hidden == "nan" else np.inf
        rec["p"][off & (np.arange(700) % 3 == 0)] = v
        rec["dout"][off & (np.arange(700) % 3 == 1)] = v
        rec["rtot"][off & (np.arange(700) % 3 == 2)] = v
    elif hidden == "receiver":
        rec["p"][off] = sim["rx_pos"][np.arange(off.sum()) % M]
    else:
        rec["mat"][off] = np.array([-1, 1 << 30, -(1 << 31), 77], np.int64)[np.arange(off.sum()) % 4].astype(np.int32)
    P = et.Paths.from_records(rec)
    ref = O.synth({k: v[~off] for k, v in rec.items()}, sim)
    flags = et.ET_SPECULAR | et.ET_DIFFRACTION | et.ET_PASSIVE | (et.ET_SYNTH_DIRECT if direct else 0)
    for what, H in _forms(et, ctx, sim, flags, P):
        assert np.all(np.isfinite(H)), what
        check_spectra(H, ref, f"{layout}, hidden {hidden}, {what}", tol=4e-6)


@pytest.mark.parametrize("layout", LAYOUTS)
def test_hidden_from_one_receiver(et, ctx, layout):
    """Per-receiver line of sight: a record on a receiver that it is hidden from counts for the others alone."""
    sim, g = _sim(*layout)
    M = len(sim["rx_pos"])
    rec = _records(g, 400, 3, M, kinds=(0, 0, 1))
    rec["rxvis"] = g.integers(1, 1 << M, 400).astype(np.uint64)
    for m in range(M):
        at = np.flatnonzero((rec["rxvis"] >> np.uint64(m)) & np.uint64(1) == 0)[:5]
        rec["p"][at] = sim["rx_pos"][m]
    sim = dict(sim, per_rx_visibility=True)
    ref = O.synth(rec, sim)
    P = et.Paths.from_records(rec)
    for what, H in _forms(et, ctx, sim, et.ET_SPECULAR | et.ET_DIFFRACTION | et.ET_PER_RX_VISIBILITY, P):
        check_spectra(H, ref, f"{layout}, hidden from one receiver, {what}", tol=4e-6)


@pytest.mark.parametrize("layout", LAYOUTS)
def test_records_of_kind_3_are_passive_at_every_receiver(et, ctx, layout):
    """(the two bits of the kind hold four values; the per-term kernel reads the fourth so)"""
    sim, g = _sim(*layout)
    rec = _records(g, 200, 3, len(sim["rx_pos"]), kinds=(0, 1))
    rec["kind"][::2] = 3
    rec["mat"][::2] = g.integers(0, 50, 100)
    P = et.Paths.from_records(rec)
    flags = et.ET_SPECULAR | et.ET_PASSIVE
    D = et.synthesize(ctx, et.Sim(sim, flags=flags | et.ET_SYNTH_DIRECT), P).cpu().numpy()
    for what, H in _forms(et, ctx, sim, flags, P):
        check_spectra(H, D, f"{layout}, kind 3, {what}", tol=8e-6)


@pytest.mark.parametrize("beta", [0.0, 1e-23, np.nan])
@pytest.mark.parametrize("layout", LAYOUTS)
def test_lobe_widths_are_the_specular_records_own(et, ctx, layout, beta):
    """Material 0 with lobes of width 0, of a width whose square underflows, and of no width at all: diffraction and passive
    records of every material, and specular ones of the others, are the oracle's all the same."""
    sim, g = _sim(*layout)
    rec = _records(g, 300, 3, len(sim["rx_pos"]), kinds=(0, 1, 1, 2))
    spec = rec["kind"] == 0
    rec["mat"][spec] = 1 + rec["mat"][spec] % 2
    ref_mix, ref_rest = O.synth(rec, sim), O.synth({k: v[~spec] for k, v in rec.items()}, sim)
    sim["lobe_beta"][0] = beta
    flags = et.ET_SPECULAR | et.ET_DIFFRACTION | et.ET_PASSIVE
    for part, ref in ((rec, ref_mix), ({k: v[~spec] for k, v in rec.items()}, ref_rest)):
        for what, H in _forms(et, ctx, sim, flags, et.Paths.from_records(part)):
            check_spectra(H, ref, f"{layout}, beta of material 0 {beta}, {what}", tol=4e-6)


@pytest.mark.parametrize("weak", [1e-4, 1e-6, 1e-8, 1e-12])
@pytest.mark.parametrize("F,Bk,Bd,direct", [(3000, 7, 0, False), (3000, 7, 3, False), (500, 4, 0, False), (130, 3, 0, False),
                                            (3000, 7, 0, True)])
def test_weak_bands_keep_their_precision(et, ctx, F, Bk, Bd, direct, weak):
    """Bands off the 64-bin blocks with coefficients from 1 down to `weak`, on paths of 1 to 65 m with the default absorption
    (up to 190 dB more in the last band than in the first): every band's own relative error, not the whole spectrum's.
    An FP32 term's exponent (below 64 with the weakest band) is rounded to 2^-19, 1.3e-6 of the term; with the
    lobe's angle and the sums 5e-6."""
    sim, g = _sim(F, Bk, Bd, seed=17)
    k = np.geomspace(1.0, weak, Bk).astype(np.float32)
    sim.update(refl_k=np.stack([np.roll(k, i) for i in range(3)]), diff_coef=np.stack([np.roll(k, -i) for i in range(3)]),
               passive_coef=k[::-1].copy(), lobe_beta=np.full((3, Bk), 1.5, np.float32), atm_a0=0.0, atm_a1=3.5e-5)
    far = g.random(500) < 0.5
    flags = et.ET_SPECULAR | et.ET_DIFFRACTION | et.ET_PASSIVE | (et.ET_SYNTH_DIRECT if direct else 0)
    for pick in (far, ~far, np.ones(500, bool)):
        rec = _records(g, 500, 3, len(sim["rx_pos"]))
        rec["rtot"] = np.where(far, g.uniform(55, 60, 500), g.uniform(0.5, 4, 500))
        # (one material: every record weak in the same band)
        rec["mat"] = np.where(rec["kind"] == 2, rec["mat"], 0)
        rec = {a: v[pick] for a, v in rec.items()}
        ref = O.synth(rec, sim)
        band = np.arange(F) * Bk // F
        for what, H in _forms(et, ctx, sim, flags, et.Paths.from_records(rec)):
            assert ctx.stats().synth_kernel == 2 and ctx.stats().synth_rows == (0 if direct else 1)
            for b in range(Bk):
                e = np.linalg.norm(H[:, band == b] - ref[:, band == b]) / np.linalg.norm(ref[:, band == b])
                assert e <= 5e-6, f"band {b} of {Bk}, {what}: {e:.2e}"


@pytest.mark.parametrize("layout", [l for l in LAYOUTS if l[2]] + [(4096, 64, 3)])
def test_gains_below_the_normal_range(et, ctx, layout):
    """Directivity gains around 1e-40 (FP32 keeps 16 bits of them, 2e-5) beside coefficients of 1e30 are gains, not nothing."""
    sim, g = _sim(*layout)
    sim["directivity"] = (sim["directivity"] * np.float32(1e-20) * np.float32(1e-20)).astype(np.float32)
    assert np.all(sim["directivity"] < 1.2e-38) and np.any(sim["directivity"] > 1e-41)
    sim.update(refl_k=sim["refl_k"] * np.float32(1e30), diff_coef=sim["diff_coef"] * np.float32(1e30))
    rec = _records(g, 300, 3, len(sim["rx_pos"]), kinds=(0, 1))
    ref = O.synth(rec, sim)
    for what, H in _forms(et, ctx, sim, et.ET_SPECULAR | et.ET_DIFFRACTION, et.Paths.from_records(rec)):
        check_spectra(H, ref, f"{layout}, gains of 1e-40, {what}", tol=1e-4)
