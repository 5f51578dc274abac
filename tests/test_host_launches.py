"""libu1ml's host side on the CPU (tests/helpers/host_hip.py): contexts of
problems at the ends of the accepted range, and what their calls launch."""
import pytest

from helpers import host_hip


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_hip.build(tmp_path_factory.mktemp("host_hip"))


@pytest.mark.parametrize("ns,nt,precision,block", [((2, 2, 2), 262144, 0, 256), ((2, 2, 2), 65536, 0, 1024),
                                                   ((2, 2, 2), 524288, 1, 256), ((64, 4, 2), 131072, 1, 1024),
                                                   ((64, 8, 2), 65536, 0, 256)])
def test_long_time_extents(so, ns, nt, precision, block):
    """Bytes of a stretch of every time slice reach 2^32 (with planes that are
    whole work-groups and with ones that are not): the tables are built, and a
    phase covers every link."""
    (grid,) = host_hip.run(so, f"""
ctx = make(u1.Spec(ensembles=[u1.Ens({ns}, {nt}, 1.0)], levels=[(2, 1, 1)], r=[1], precision={precision}))
ok(L.u1ml_set_block(ctx, {block}))
ok(L.u1ml_init_links(ctx, u1.HOT))
launches()
ok(L.u1ml_phase(ctx, u1.OVERRELAX, 3, 0, 0, 0))
(l,) = launches()
assert l[0] == "k_update" and l[2][0] == {block}, l
put(l[1][0])
ok(L.u1ml_destroy(ctx))
""")
    links = ns[0] // 2 * ns[1] * ns[2] * nt
    assert grid * block >= links


@pytest.mark.parametrize("kw", [dict(n=16384, form=1, r=[1, 2, 3], probes=126, comps=1),
                                dict(n=16384, form=2, r=[1, 2, 3, 1], probes=14, comps=6),
                                dict(n=3000, L=16, form=2, r=[1], probes=62, comps=1)])
def test_many_sums(so, kw):
    """Batches whose sums, a wave or a work-group each, are more than a grid
    holds: estimates of many probes on thousands of small lattices."""
    host_hip.run(so, f"""
kw = {kw}
N = kw.get("L", 4)
probes = [(l, a, b, m) for l in range(1 - N, N) for m in (0, 1) for a, b in
          ([(0, 0)] if kw["probes"] < 100 else [(a, b) for a in (-1, 0, 1) for b in (-1, 0, 1)])]
spec = u1.Spec(ensembles=[u1.Ens((N, N, N), 4, 1.0, key_id=i) for i in range(kw["n"])], levels=[(2, 1, 0)], r=kw["r"],
               probes=probes[: kw["probes"]], comps=list(range(kw["comps"])), form=kw["form"])
ctx = make(spec)
ok(L.u1ml_set_lanes(ctx, 1))
ok(L.u1ml_init_links(ctx, u1.HOT))
launches()
ok(L.u1ml_multilevel(ctx), ctx)
assert any(l[0] == ("k_product_final" if kw["form"] == 1 else "k_spec_final") for l in launches())
ok(L.u1ml_destroy(ctx))
""", timeout=300)


@pytest.mark.parametrize("tau", [65536, 131072])
def test_multihit_of_thick_slabs(so, tau):
    """More time slices in a slab than a grid has along its second axis."""
    host_hip.run(so, f"""
ctx = make(u1.Spec(ensembles=[u1.Ens((2, 2, 2), 131072, 1.0)], levels=[({tau}, 1, 0)], r=[1], multihit=True))
ok(L.u1ml_init_links(ctx, u1.HOT))
ok(L.u1ml_multilevel(ctx), ctx)
assert "k_multihit" in [l[0] for l in launches()]
ok(L.u1ml_destroy(ctx))
""")


@pytest.mark.parametrize("call", ["plan", "create", "set_block", "set_lanes"])
def test_no_exception_leaves_the_library(so, call):
    """Out of host memory: U1ML_ENOMEM with a message, and a context whose call
    failed goes on as it was."""
    host_hip.run(so, f"""
import resource
call = {call!r}
ns, nt, n = ((2, 2, 2), 2, 2000000) if call == "plan" else ((8, 4, 4), 300000, 3)
spec = u1.Spec(ensembles=[u1.Ens(ns, nt, 1.0, key_id=i) for i in range(n)], levels=[(60000 if n == 3 else 2, 1, 0)], r=[1])
p = spec.struct()
info = u1._PlanInfo()
h = C.c_void_p()
if call not in ("plan", "create"):
    h = make(spec)
    ok(L.u1ml_set_lanes(h, 1))
    ok(L.u1ml_init_links(h, u1.HOT))
    launches()
    ok(L.u1ml_phase(h, u1.OVERRELAX, 3, 0, 0, 0))
    before = launches()
used = int(open("/proc/self/statm").read().split()[0]) * 4096
resource.setrlimit(resource.RLIMIT_AS, (used + (64 << 20), -1))
st = (L.u1ml_plan(C.byref(p), C.byref(info)) if call == "plan" else
      L.u1ml_create(C.byref(p), C.c_void_p(1 << 40), 1 << 50, None, C.byref(h)) if call == "create" else
      L.u1ml_set_block(h, 64) if call == "set_block" else L.u1ml_set_lanes(h, 3))
resource.setrlimit(resource.RLIMIT_AS, (-1, -1))
assert st == 2, st
assert b"allocation" in L.u1ml_last_error(h if call[0] == "s" else None)
if call in ("plan", "create"):
    assert not h.value
else:
    ok(L.u1ml_phase(h, u1.OVERRELAX, 3, 0, 0, 0))
    assert launches() == before
    n_lanes = C.c_int()
    ok(L.u1ml_get_lanes(h, C.byref(n_lanes)))
    assert n_lanes.value == 1
    ok(L.u1ml_multilevel(h))
    ok(L.u1ml_destroy(h))
""")


def test_planning_time_of_equal_lattices():
    """A plan of 2048 equal lattices takes no more than ten times that of 2048
    lattices whose sweeps run in LDS, for which no tiles are looked for."""
    import ctypes as C
    import time

    from paper_1309_3859_amd import u1ml as u1

    def seconds(n, ns, nt):
        p = u1.Spec(ensembles=[u1.Ens(ns, nt, 1.0, key_id=i) for i in range(n)], levels=[(2, 1, 1)], r=[1]).struct()
        info = u1._PlanInfo()
        best = 1e9
        for _ in range(5):
            t = time.process_time()
            assert u1.lib().u1ml_plan(C.byref(p), C.byref(info)) == 0
            best = min(best, time.process_time() - t)
        return best

    base = seconds(2048, (4, 4, 4), 4)
    assert seconds(2048, (8, 8, 8), 16) < 10 * base
    assert seconds(512, (16, 16, 16), 8) < 10 * base


@pytest.mark.parametrize("ns,nt,levels", [((24, 24, 24), 8, [(2, 3, 1)]), ((12, 12, 12), 12, [(4, 2, 1), (2, 2, 1)]),
                                          ((4, 4, 4), 4, [(2, 2, 1)]), ((32, 32, 32), 32, [(2, 1, 1)])])
@pytest.mark.parametrize("n_or", [0, 1, 2, 3])
def test_second_link_buffer_only_where_it_is_used(so, ns, nt, levels, n_or):
    """The other link buffer is reserved, and the frozen links copied to it, only
    where sweeps update both parities of a spatial direction in one launch."""
    second, names = host_hip.run(so, f"""
spec = u1.Spec(ensembles=[u1.Ens({ns}, {nt}, 1.0)], levels={levels}, r=[1], n_or={n_or}, precision=u1.FP32)
p = u1.plan(spec)
put(p["ws_bytes"] - sum(p[k + "_bytes"] for k in ("link", "history", "average", "outer", "result", "scratch", "spectral")))
ctx = make(spec)
ok(L.u1ml_init_links(ctx, u1.HOT))
launches()
ok(L.u1ml_sweeps(ctx, 1))
ok(L.u1ml_multilevel(ctx))
put([l[4] for l in launches()])
ok(L.u1ml_destroy(ctx))
""")
    pairs = [n for n in names if "k_pair" in n]
    assert (second > 0) == bool(pairs)
    if not any("ELi%dEE" % mu in n for n in pairs for mu in range(3)):
        assert not any("k_mirror" in n for n in names)


@pytest.mark.parametrize("n,ns,nt,precision,full,slab", [
    (1, (24, 24, 24), 8, 1, "xyzt", "xyzt"),   # us per sweep with none / all paired: full 89 / 78, inside slabs 85 / 63
    (1, (24, 24, 24), 8, 0, "t", "xyzt"),      # 122 / 145, 118 / 101
    (1, (24, 24, 24), 12, 0, "", None),        # 149 / 215
    (1, (8, 8, 8), 512, 0, "t", None),         # 148 / 208, t alone 143
    (1, (6, 6, 6), 2048, 1, "t", None),        # 121 / 146, t alone 116
    (16, (12, 12, 12), 8, 0, "", None),        # 144 / 222
    (1, (48, 48, 48), 4, 0, "", ""),           # 220 / 396, 165 / 214
    (1, (32, 32, 32), 8, 1, None, "xyz"),      # inside slabs 84 / 74.5, t alone 85, without t 73.9
])
def test_directions_paired_where_it_is_faster(so, n, ns, nt, precision, full, slab):
    """Which directions a sweep updates in one launch for both parities, on
    lattices where an MI355X was timed with every direction either way."""
    got = host_hip.run(so, f"""
ctx = make(u1.Spec(ensembles=[u1.Ens({ns}, {nt}, 1.0, key_id=i) for i in range({n})], levels=[(2, 1, 1)], r=[1],
                   precision={precision}))
ok(L.u1ml_set_lanes(ctx, 1))
ok(L.u1ml_init_links(ctx, u1.HOT))
launches()
for call in (lambda: L.u1ml_sweeps(ctx, 1), lambda: L.u1ml_multilevel(ctx)):
    ok(call())
    names = [l[4] for l in launches()]
    put("".join("xyzt"[mu] for mu in range(4) if any("k_pair" in m and "ELi%dEE" % mu in m for m in names)))
ok(L.u1ml_destroy(ctx))
""")
    assert full is None or got[0] == full
    assert slab is None or got[1] == slab


@pytest.mark.parametrize("n,ns,nt,precision,full,slab", [
    # us per sweep in LDS / otherwise
    (1, (4, 4, 4), 4, 0, True, True),
    (4096, (4, 4, 4), 8, 0, True, True),     # full 528 / 582, slabs 513 / 518
    (256, (8, 8, 8), 4, 0, False, True),     # slabs 124 / 151
    (512, (8, 8, 8), 4, 0, False, False),    # 245 / 223
    (2048, (8, 8, 8), 4, 0, False, False),   # 1056 / 944
    (512, (6, 6, 6), 8, 0, False, False),    # 258 / 219
    (768, (6, 6, 6), 4, 0, True, True),      # full 240 / 280, slabs 193 / 227
    (1024, (6, 6, 6), 4, 0, False, False),   # 323 / 306, 256 / 221
    (1024, (4, 6, 4), 8, 0, False, False),   # 326 / 301, 250 / 222
    (1024, (2, 4, 4), 16, 0, True, False),   # 154 / 214, 259 / 176
    (2048, (2, 4, 4), 16, 1, True, False),   # 97 / 162, 164 / 137
    (1024, (8, 8, 16), 2, 1, True, True),    # full 208 / 217
    (3072, (8, 8, 16), 2, 1, False, True),   # full 617 / 578, slabs 464 / 490
])
def test_sweeps_in_lds_where_it_is_faster(so, n, ns, nt, precision, full, slab):
    """Which sweeps run in LDS, on batches where an MI355X was timed with both."""
    got = host_hip.run(so, f"""
ctx = make(u1.Spec(ensembles=[u1.Ens({ns}, {nt}, 1.0, key_id=i) for i in range({n})], levels=[(2, 1, 1)], r=[1],
                   precision={precision}))
ok(L.u1ml_init_links(ctx, u1.HOT))
launches()
for call in (lambda: L.u1ml_sweeps(ctx, 1), lambda: L.u1ml_multilevel(ctx)):
    ok(call())
    put(any(l[0] == "k_slab" for l in launches()))
ok(L.u1ml_destroy(ctx))
""")
    assert got == [full, slab]


@pytest.mark.parametrize("n,ns,nt,precision,lanes", [
    # us per sweep, full / inside slabs, with 1 and with 2 lanes
    (8, (24, 24, 24), 8, 1, 1),     # 147 / 111, 158 / 133
    (256, (8, 8, 8), 8, 1, 2),      # 160 / 72, 154 / 74
    (32, (16, 16, 16), 8, 1, 2),    # 161 / 120, 151 / 119
    (8, (24, 24, 24), 4, 0, 1),     # 214 / 158, 193 / 169
    (16, (16, 16, 16), 8, 0, 2),    # 218 / 160, 195 / 154
])
def test_lanes_where_two_are_faster(so, n, ns, nt, precision, lanes):
    (got,) = host_hip.run(so, f"""
ctx = make(u1.Spec(ensembles=[u1.Ens({ns}, {nt}, 1.0, key_id=i) for i in range({n})], levels=[(2, 1, 1)], r=[1],
                   precision={precision}))
k = C.c_int()
ok(L.u1ml_get_lanes(ctx, C.byref(k)))
put(k.value)
ok(L.u1ml_destroy(ctx))
""")
    assert got == lanes


@pytest.mark.parametrize("kw", [
    dict(ns=(4, 4, 4), nt=4, levels=[(2, 300, 1)]), dict(ns=(24, 24, 24), nt=8, levels=[(2, 50, 1)], precision=1),
    dict(ns=(24, 24, 24), nt=8, levels=[(2, 20, 2)], n_or=2), dict(ns=(24, 24, 24), nt=8, levels=[(2, 20, 2)], n_or=0),
    dict(ns=(32, 32, 32), nt=8, levels=[(4, 5, 3), (2, 10, 1)], precision=1, probes=1, form=1),
    dict(ns=(32, 32, 32), nt=8, levels=[(4, 5, 3), (2, 10, 1)], precision=1, probes=1, form=2),
    dict(ns=(8, 8, 8), nt=8, levels=[(4, 5, 130), (2, 10, 70)], multihit=True, probes=9, form=2),
    dict(ns=(48, 48, 48), nt=12, levels=[(4, 3, 0), (2, 4, 1)], precision=1, n=3),
    dict(ns=(12, 12, 12), nt=12, levels=[(2, 6, 2), (2, 5, 1)], update=1)])
def test_planned_launch_count(so, kw):
    """u1ml_plan's launches_per_config against the launches of a configuration on
    one lane: never fewer, and more by what it grants per level, configuration
    and ensemble (of which a form uses a part) only."""
    planned, issued = host_hip.run(so, f"""
kw = dict({kw})
n, k = kw.pop("n", 1), kw.pop("probes", 0)
ns, nt = kw.pop("ns"), kw.pop("nt")
spec = u1.Spec(ensembles=[u1.Ens(ns, nt, 1.0, key_id=i) for i in range(n)], r=[1, 2],
               probes=[(0, a, b, 1) for a in (0, 1, -1) for b in (0, 1, -1)][:k], comps=[0, 3] if k else [], **kw)
put(u1.plan(spec)["launches_per_config"])
ctx = make(spec)
ok(L.u1ml_set_lanes(ctx, 1))
ok(L.u1ml_init_links(ctx, u1.HOT))
launches()
ok(L.u1ml_multilevel(ctx), ctx)
put(len(launches()))
ok(L.u1ml_destroy(ctx))
""")
    n_outer = kw["levels"][0][1] if len(kw["levels"]) == 2 else 1
    assert issued <= planned <= issued + 2 * 8 * n_outer + 10 + 5 * kw.get("n", 1)


@pytest.mark.parametrize("ns,nt,n_or,kernels", [((4, 4, 4), 4, 3, {"k_slab"}), ((24, 24, 24), 8, 3, {"k_mirror", "k_pair"}),
                                                ((24, 24, 24), 8, 2, {"k_mirror", "k_pair", "k_update"}),
                                                ((64, 64, 64), 8, 3, {"k_update"})])
def test_autotune_times_the_sweeps_that_run(so, ns, nt, n_or, kernels):
    """The launches that autotune times are those of a configuration's sweeps;
    the work-group size stays where none of them depends on it."""
    tuned, run, chosen = host_hip.run(so, f"""
ctx = make(u1.Spec(ensembles=[u1.Ens({ns}, {nt}, 1.0)], levels=[(2, 1, 1)], r=[1], n_or={n_or}, precision=u1.FP32))
ok(L.u1ml_init_links(ctx, u1.HOT))
launches()
rep = u1._TuneReport()
ok(L.u1ml_autotune(ctx, C.byref(rep)))
kinds = ("k_slab", "k_pair", "k_mirror", "k_update")
put(sorted(set(l[0] for l in launches()) & set(kinds)))
ok(L.u1ml_multilevel(ctx))
put(sorted(set(l[0] for l in launches()) & set(kinds)))
put(rep.chosen_block)
ok(L.u1ml_destroy(ctx))
""")
    assert set(tuned) == set(run) == kernels
    if "k_update" not in kernels:
        assert chosen == 256
