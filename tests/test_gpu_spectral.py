"""Parity of the spectral form of the insertion estimators (plane transforms
over the plane orthogonal to the charge axis; two levels replay each
configuration), through the C ABI.

* against the history form on the same device trajectory (same links, same
  counters), one and two levels, several axes, probes of both modes and
  several probe groups, plane extents taking every radix of the plane FFT and
  extents taking the direct sums: every estimate within FP64 rounding of the
  contraction order;
* after a two-level configuration the links and counters equal those of the
  history form (the replay restores the start and repeats the trajectory);
* against the oracle's independent FP64 chain (heatbath-only trajectories,
  whose GPU/oracle link agreement is at the 1e-12 level);
* the largest preset's full 441-probe map at full size (48^3 x 12, FP32
  links), one measurement without updates, sampled probes against the oracle.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle as O
    from paper_1309_3859_amd import configs, u1ml

    u1ml.lib()
    O.build()
    return u1ml, O, configs


def _disk(rad, mode=1, l=0):
    return [(l, p1, p2, mode) for p1 in range(-rad, rad + 1) for p2 in range(-rad, rad + 1) if p1 * p1 + p2 * p2 <= rad * rad]


def _run(u1, spec, form, start_seed_sweeps=2):
    spec.form = form
    ctx = u1.Context(spec)
    assert ctx.plan["form"] == (u1.FORM_SPECTRAL if form == u1.FORM_SPECTRAL else u1.FORM_HISTORY)
    ctx.init_links(u1.HOT)
    ctx.sweeps(start_seed_sweeps)
    ctx.multilevel()
    res = ctx.results()[0]
    links = [ctx.links(e) for e in range(len(spec.ensembles))]
    cnt = [ctx.counter(e) for e in range(len(spec.ensembles))]
    return res, links, cnt


def _compare(spec, ra, rb, rel):
    for e in range(len(spec.ensembles)):
        a, b = spec.unpack(ra[e]), spec.unpack(rb[e])
        scale = max(1.0, float(np.abs(a["CO"]).max()))
        d = float(np.abs(a["CO"] - b["CO"]).max())
        say("  ensemble", e, "max |dCO|", d, "scale", scale, "max |dC|", float(np.abs(a["C"] - b["C"]).max()))
        assert d <= rel * scale
        assert np.allclose(a["C"], b["C"], rtol=0, atol=1e-14)
        assert np.allclose(a["vac_sq"], b["vac_sq"], rtol=0, atol=1e-14)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_spectral_one_level_matches_history(env, prec):
    u1, O, _ = env
    mk = lambda: u1.Spec(ensembles=[u1.Ens((6, 6, 6), 4, 1.0, seed=11), u1.Ens((8, 6, 6), 6, 0.9, seed=12, key_id=3)],
                         levels=[(2, 3, 1)], r=[1, 2, 3], dirs=[0, 1, 2],
                         probes=_disk(2) + [(1, 0, 1, 0), (-1, 1, 0, 0), (0, -2, 1, 0)], comps=list(range(6)),
                         precision=u1.FP64 if prec == "fp64" else u1.FP32, n_or=3)
    say("one level", prec)
    rh, lh, ch = _run(u1, mk(), u1.FORM_HISTORY)
    rs, ls, cs = _run(u1, mk(), u1.FORM_SPECTRAL)
    for a, b in zip(lh, ls):
        assert np.array_equal(a, b)
    assert ch == cs
    _compare(mk(), rh, rs, 1e-12)


def test_spectral_transform_sizes_match_history(env):
    """Plane extents that take every radix of the plane FFT (4, 2, 3, 5) and
    extents with a prime factor above 5 (14), which take the direct sums."""
    u1, O, _ = env
    mk = lambda: u1.Spec(ensembles=[u1.Ens((6, 10, 14), 4, 1.0, seed=13), u1.Ens((12, 20, 8), 4, 0.95, seed=14, key_id=2)],
                         levels=[(2, 2, 1)], r=[1, 3], dirs=[0, 1, 2], probes=_disk(1) + [(2, 1, -1, 0)],
                         comps=[0, 2, 4], precision=u1.FP64, n_or=2)
    say("transform sizes")
    rh, lh, ch = _run(u1, mk(), u1.FORM_HISTORY)
    rs, ls, cs = _run(u1, mk(), u1.FORM_SPECTRAL)
    for a, b in zip(lh, ls):
        assert np.array_equal(a, b)
    _compare(mk(), rh, rs, 1e-12)


@pytest.mark.parametrize("n_comp", [1, 2, 3, 4, 5, 6])
def test_spectral_sums_of_every_component_count(env, n_comp):
    """Each number of components is a kernel of its own; 25 separations take
    two rounds of its work-items, 26 positions end in a partial buffer and
    planes of 36 sites in a partial tile.  Both forms sum the same products
    (|T|, |O| <= 1) in FP64: the shared bar of this file."""
    u1, O, _ = env
    mk = lambda: u1.Spec(ensembles=[u1.Ens((26, 6, 6), 4, 1.0, seed=17)], levels=[(2, 2, 1)], r=list(range(1, 26)),
                         dirs=[0], probes=_disk(1) + [(3, 1, 0, 0)], comps=list(range(6))[6 - n_comp:],
                         precision=u1.FP64, n_or=1)
    say("components", n_comp)
    rh, _, _ = _run(u1, mk(), u1.FORM_HISTORY)
    rs, _, _ = _run(u1, mk(), u1.FORM_SPECTRAL)
    _compare(mk(), rh, rs, 1e-12)


@pytest.mark.parametrize("n_probe", [1, 512, 513])
def test_spectral_probe_counts(env, n_probe):
    """One work-item reads off one probe: a single probe, a full work-group
    and one more (a second pass), up to seven groups, axes of unequal
    planes.  The shared bar of this file."""
    u1, O, _ = env
    probes = [(i // 81 - 3, i % 9 - 4, i // 9 % 9 - 4, 1) for i in range(n_probe)]
    mk = lambda: u1.Spec(ensembles=[u1.Ens((12, 14, 10), 4, 1.0, seed=19)], levels=[(2, 2, 1)], r=[1, 2],
                         dirs=[0, 1, 2], probes=probes, comps=[1, 5], precision=u1.FP64, n_or=1)
    say("probes", n_probe)
    rh, _, _ = _run(u1, mk(), u1.FORM_HISTORY)
    rs, _, _ = _run(u1, mk(), u1.FORM_SPECTRAL)
    _compare(mk(), rh, rs, 1e-12)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("side", [12, 16, 18, 20, 24, 30, 32, 36, 40, 48, 60, 64])
def test_spectral_square_planes(env, side, prec):
    """Each side that has a transform in registers, both link types; the
    extent along the charge axis differs from the planes' sides.  The shared
    bar of this file."""
    u1, O, _ = env
    mk = lambda: u1.Spec(ensembles=[u1.Ens((6, side, side), 4, 1.0, seed=23)], levels=[(2, 2, 1)], r=[1, 2],
                         dirs=[0], probes=_disk(2), comps=[0, 3], precision=u1.FP64 if prec == "fp64" else u1.FP32,
                         n_or=1)
    say("square planes", side, prec)
    rh, _, _ = _run(u1, mk(), u1.FORM_HISTORY)
    rs, _, _ = _run(u1, mk(), u1.FORM_SPECTRAL)
    _compare(mk(), rh, rs, 1e-12)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_spectral_two_levels_replay_matches_history(env, prec):
    u1, O, _ = env
    mk = lambda: u1.Spec(ensembles=[u1.Ens((6, 6, 6), 8, 1.0, seed=21)], levels=[(4, 2, 1), (2, 3, 1)], r=[1, 2],
                         dirs=[0, 2], probes=_disk(1) + [(2, 1, -1, 0)], comps=[0, 1, 3, 5],
                         precision=u1.FP64 if prec == "fp64" else u1.FP32, n_or=2)
    say("two levels", prec)
    rh, lh, ch = _run(u1, mk(), u1.FORM_HISTORY)
    rs, ls, cs = _run(u1, mk(), u1.FORM_SPECTRAL)
    for a, b in zip(lh, ls):
        assert np.array_equal(a, b)  # the replay left the links where one pass leaves them
    assert ch == cs
    _compare(mk(), rh, rs, 1e-12)


def test_spectral_two_levels_against_oracle(env):
    u1, O, _ = env
    spec = u1.Spec(ensembles=[u1.Ens((4, 4, 4), 8, 1.0, seed=31)], levels=[(4, 2, 1), (2, 2, 1)], r=[1, 2],
                   dirs=[0, 1], probes=_disk(1) + [(1, 1, 1, 0)], comps=list(range(6)), precision=u1.FP64, n_or=0,
                   form=u1.FORM_SPECTRAL)
    ctx = u1.Context(spec)
    ctx.init_links(u1.HOT)
    ctx.sweeps(1)
    th0, cnt = ctx.links(0), ctx.counter(0)
    ctx.multilevel()
    got = spec.unpack(ctx.results()[0][0])
    e = spec.ensembles[0]
    ref = O.Lattice(4, list(e.ns) + [e.nt], e.beta, seed=e.seed, key_id=e.key_id)
    ref.set_links(th0)
    ref.counter = cnt
    ospec = O.MLSpec(levels=spec.levels, r=spec.r, dirs=spec.dirs, probes=spec.probes, comps=spec.comps, n_or=0)
    want = ospec.unpack(ref.multilevel(ospec))
    scale = max(1.0, float(np.abs(want["CO"]).max()))
    d = float(np.abs(got["CO"] - want["CO"]).max())
    say("vs oracle: max |dCO|", d, "scale", scale, "max |dC|", float(np.abs(got["C"] - want["C"]).max()))
    assert d < 1e-9 * scale
    assert np.max(np.abs(got["C"] - want["C"])) < 1e-10
    assert np.max(np.abs(got["vac_sq"] - want["vac_sq"])) < 1e-10


def test_full_map_of_largest_preset_sampled(env):
    """48^3 x 12, two levels, 441 probes x 19 r x 6 components in the spectral
    form at full size; one measurement without updates, so the estimates are
    functions of the links alone; sampled probes and separations against the
    oracle on the same links."""
    u1, O, configs = env
    spec, sched = configs.c5_largest(n_outer=1, n_inner=1, full_map=True)
    spec.levels = [(4, 1, 0), (2, 1, 0)]
    ctx = u1.Context(spec)
    say("C5 full map: form", ctx.plan["form"], "workspace", ctx.plan["ws_bytes"])
    assert ctx.plan["form"] == u1.FORM_SPECTRAL
    ctx.init_links(sched["start"])
    ctx.sweeps(2)
    ctx.multilevel()
    got = spec.unpack(ctx.results()[0][0])
    pick_p = [spec.probes.index(p) for p in [(0, 0, 0, 1), (0, 12, 0, 1), (0, 0, -12, 1), (0, 8, 8, 1),
                                              (0, -5, 7, 1)]]
    pick_r = [0, 9, 18]  # r = 2, 11, 20
    e = spec.ensembles[0]
    ref = O.Lattice(4, list(e.ns) + [e.nt], e.beta, seed=e.seed, key_id=e.key_id)
    ref.set_links(ctx.links(0))
    ospec = O.MLSpec(levels=spec.levels, r=[spec.r[i] for i in pick_r], dirs=spec.dirs,
                     probes=[spec.probes[i] for i in pick_p], comps=spec.comps, n_or=spec.n_or)
    want = ospec.unpack(ref.multilevel(ospec))
    sub = got["CO"][np.ix_(pick_r, pick_p)]
    scale = max(1.0, float(np.abs(want["CO"]).max()))
    d = float(np.abs(sub - want["CO"]).max())
    say("  sampled max |dCO|", d, "scale", scale)
    assert d < 2e-5 * scale
    assert np.max(np.abs(got["C"][pick_r] - want["C"])) < 1e-12


@pytest.mark.parametrize("ns,dirs", [((4, 24, 24), [0]), ((6, 10, 14), [0, 2]), ((2, 64, 64), [0]), ((2, 2, 106), [0])],
                         ids=["24x24", "two axes", "64x64", "2x106"])
def test_probe_sums_round_no_more_than_term_by_term(env, ns, dirs):
    """The estimates against their definition, the sum over slabs and over the
    plane of the accumulated spectra F(k) e^{2 pi i k p}, read back from the
    workspace and summed in extended precision: root-mean-square error over the
    probes, no larger than that of the plain sum, every term formed in FP64
    ((w1 w2) F / (n1 n2)) and added without error.  Slabs alike (links constant
    in time), so that their spectra add up."""
    u1, O, _ = env
    LD, CLD = np.longdouble, np.clongdouble
    nt, R, comps = 12, 1, [0, 3]
    rng = np.random.default_rng(5)
    p1s = range(1 - min((ns[(d + 1) % 3] + 1) // 2 for d in dirs), min((ns[(d + 1) % 3] + 1) // 2 for d in dirs))
    p2s = range(1 - min((ns[(d + 2) % 3] + 1) // 2 for d in dirs), min((ns[(d + 2) % 3] + 1) // 2 for d in dirs))
    probes = [(0, a, b, 1) for a in p1s for b in p2s]
    if len(probes) > 300:
        probes = [probes[i] for i in rng.choice(len(probes), 300, replace=False)]
    spec = u1.Spec(ensembles=[u1.Ens(ns, nt, 1.0)], levels=[(2, 1, 0)], r=[1], dirs=dirs, probes=probes, comps=comps,
                   precision=u1.FP64, form=u1.FORM_SPECTRAL)
    ctx = u1.Context(spec)
    nsig = ns[0] * ns[1] * ns[2]
    ctx.set_links(np.tile(rng.uniform(-np.pi, np.pi, 4 * nsig), nt))
    say("probe sums", ns, dirs, len(probes))
    ctx.multilevel()
    got = spec.unpack(ctx.results()[0][0])["CO_mant"][0]  # [probe, comp, kind]

    pl, nd, S, nc = ctx.plan, len(dirs), nt // 2, len(comps)
    up = lambda n: (n + 255) // 256 * 256
    rest = sum(pl[k] for k in ("link_bytes", "history_bytes", "average_bytes", "outer_bytes", "result_bytes",
                               "spectral_bytes", "scratch_bytes"))
    second = pl["ws_bytes"] - rest  # the other link buffer, where sweeps use one
    assert second in (0, pl["link_bytes"])
    off = second + rest - pl["scratch_bytes"] - pl["spectral_bytes"]
    off += up(16 * nd * R * S * nsig) + up(16 * nd * S * R * nsig) + up(16 * nd * S * 12 * nsig)  # G and the spectra
    n12max = max(nsig // ns[d] for d in dirs)
    size = nd * S * R * nc * 2 * n12max * 16
    F = ctx.ws[off: off + size].cpu().numpy().view(np.complex128).reshape(nd, S, R, nc, 2, n12max)

    exact = np.zeros((len(probes), nc, 2), CLD)
    plain = np.zeros((len(probes), nc, 2), CLD)
    turn = 2 * LD(np.arctan2(LD(0), LD(-1)))
    for i, d in enumerate(dirs):
        n1, n2 = ns[(d + 1) % 3], ns[(d + 2) % 3]
        f = F[i, :, 0, :, :, : n1 * n2].reshape(S, nc, 2, n1, n2)
        fs = f.sum(axis=0, dtype=CLD)
        # the twiddles' arguments 2 j / n are formed in FP64, in the estimates as here
        arg = lambda n: LD(0.5) * turn * (2.0 * np.arange(n) / n).astype(LD)
        tw = lambda n: [np.cos(arg(n)).astype(np.float64), np.sin(arg(n)).astype(np.float64)]
        t1, t2 = tw(n1), tw(n2)
        for k, (_, a, b, _) in enumerate(probes):
            j1, j2 = (np.arange(n1) * a) % n1, (np.arange(n2) * b) % n2
            w1, w2 = t1[0][j1] + 1j * t1[1][j1], t2[0][j2] + 1j * t2[1][j2]
            exact[k] += (fs * (w1.astype(CLD)[:, None] * w2[None, :])).sum(axis=(-2, -1)) / (n1 * n2)
            w = w1[:, None] * w2[None, :]
            inv = 1.0 / (n1 * n2)
            t = np.empty(f.shape, np.complex128)
            t.real = (f.real * w.real - f.imag * w.imag) * inv
            t.imag = (f.real * w.imag + f.imag * w.real) * inv
            plain[k] += t.sum(axis=(0, -2, -1), dtype=CLD)
    scale = 1.0 / (float(nsig) * nd * nt * 1.0)
    rms = lambda x: float(np.sqrt(np.mean(np.abs((x - exact * LD(scale)) / scale) ** 2)))
    mine, ref = rms(got.astype(CLD)), rms(plain.astype(np.complex128) * scale)
    norm = float(np.abs(F).sum() / (n12max * nc * 2))
    say("  rms error / sum of |terms|: estimates", mine / norm, "term by term", ref / norm)
    assert np.abs(got - exact.astype(np.complex128) * scale).max() < 1e-13 * norm * scale
    assert mine <= ref
