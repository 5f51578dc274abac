"""Update kernels at the sizes where their work split can go wrong: slices
that do not fill a work-group, work-groups that start inside a row or cross
rows and planes, rows longer than a work-group, extents of 2."""
import itertools

import numpy as np
import pytest

from helpers.inputs import random_links
from helpers.stats import circ_dist

SHAPES = [((2, 2, 2), 2), ((6, 10, 14), 6), ((20, 6, 2), 4), ((2, 22, 10), 2), ((160, 2, 4), 4)]


def test_small_quotients_are_exact():
    """The index decode's quotient, (a + 1/2) (1/b) in FP32 truncated, equals
    a div b for 0 <= a < b + 2^10, b <= 2^22: every b below 2^11, and larger
    ones around the values where a quotient steps."""
    f = np.float32
    for b in itertools.chain(range(1, 2048), [3 * 2**k + d for k in range(10, 21) for d in (-1, 0, 1)], [2**22 - 1, 2**22]):
        a = np.arange(max(0, b - 4), b + 1024) if b > 4096 else np.arange(b + 1024)
        q = ((a.astype(f) + f(0.5)) * (f(1) / f(b))).astype(np.int64)
        assert np.array_equal(q, a // b), b


@pytest.mark.gpu
@pytest.mark.parametrize("ns,nt", SHAPES)
def test_overrelaxation_matches_oracle(ns, nt):
    """FP64, every direction and parity from identical links.  A phase turns
    an angle by 2 arg A, so its error is twice that of the staple sum A over
    |A|: six terms whose arguments (below 3 pi) are rounded twice, 1.8e-15
    each, on either side, 2.2e-14; with the rounding of the turn itself the
    error times |A| stays below 5.4e-14, asserted as 1e-13."""
    import bench
    from oracle import oracle as O
    from paper_1309_3859_amd import u1ml

    V = int(np.prod(ns)) * nt
    spec = u1ml.Spec(ensembles=[u1ml.Ens(ns, nt, 1.1, seed=7, key_id=1)], levels=[(2, 1, 1)], r=[1])
    ctx = u1ml.Context(spec)
    ref = O.Lattice(4, list(ns) + [nt], 1.1, seed=7, key_id=1)
    th0 = random_links(V, 5)
    size = bench.staple_abs(th0, ns, nt).reshape(-1)
    for mu, p, tau in itertools.product(range(4), (0, 1), (0, 2)):
        print("phase", ns, nt, mu, p, tau, flush=True)
        ctx.set_links(th0)
        ref.set_links(th0)
        ctx.phase(1, mu, p, tau)
        ref.phase(1, mu, p, tau)
        d = circ_dist(ctx.links(0), ref.links())
        assert (d * size).max() < 1e-13


@pytest.mark.gpu
@pytest.mark.parametrize("ns,nt", SHAPES)
@pytest.mark.parametrize("precision", [0, 1])
def test_work_group_size_changes_no_bit(ns, nt, precision):
    from paper_1309_3859_amd import u1ml

    spec = u1ml.Spec(ensembles=[u1ml.Ens(ns, nt, 1.1, seed=7, key_id=1)], levels=[(2, 1, 1)], r=[1],
                     precision=precision)
    got = []
    for block in (64, 256, 1024):
        ctx = u1ml.Context(spec)
        ctx.set_block(block)
        ctx.init_links(u1ml.HOT)
        for kind, mu, p, tau in itertools.product((0, 1, 2), range(4), (0, 1), (0, 2)):
            ctx.phase(kind, mu, p, tau, pass_offset=mu)
        got.append(ctx.links(0))
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])


# slabs of one, two and three inner layers, extents of 2, tiles that do not
# divide the extents, rows of 1 .. 40 half sites, two levels, odd and even
# numbers of passes, slabs of 512 and 1024 links a phase (the most that sweeps
# in LDS take) and just fewer
RUNS = [((4, 4, 4), 4, [(2, 2, 1)], 3), ((2, 2, 2), 2, [(2, 2, 2)], 3), ((24, 24, 24), 4, [(2, 1, 1)], 3),
        ((10, 14, 6), 12, [(4, 2, 1), (2, 2, 1)], 2), ((18, 2, 22), 6, [(3, 2, 1)], 1), ((80, 6, 10), 8, [(4, 1, 1)], 0),
        ((2, 26, 14), 8, [(8, 1, 1), (4, 2, 1)], 3), ((8, 8, 8), 4, [(2, 2, 3)], 3), ((6, 8, 10), 4, [(2, 2, 1)], 3),
        ((6, 8, 12), 12, [(6, 1, 2), (2, 2, 1)], 2), ((2, 4, 6), 24, [(24, 1, 1)], 3)]


@pytest.mark.gpu
@pytest.mark.parametrize("ns,nt,levels,n_or", RUNS)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("update", [0, 1])
def test_sweeps_equal_their_phases(ns, nt, levels, n_or, precision, update):
    """Sweeps and configurations, however many phases a launch does, leave the
    links that one launch per phase leaves, bit for bit, on a batch of the
    lattice and of one half its time extent."""
    from paper_1309_3859_amd import u1ml

    print("run", ns, nt, levels, n_or, precision, update, flush=True)
    ens = [u1ml.Ens(ns, nt, 1.05, seed=3, key_id=j) for j in range(2)]
    if nt % 4 == 0 and nt // 2 % levels[0][0] == 0:
        ens.append(u1ml.Ens(ns, nt // 2, 0.9, seed=3, key_id=2))
    spec = u1ml.Spec(ensembles=ens, levels=levels, r=[1], precision=precision, n_or=n_or, update=update,
                     metro_delta=0.7)

    def sweep(ctx, tau, offset):
        for k in range(1 + n_or):
            kind = (u1ml.METROPOLIS if update else u1ml.HEATBATH) if k == 0 else u1ml.OVERRELAX
            for mu, p in itertools.product(range(4), (0, 1)):
                ctx.phase(kind, mu, p, tau, offset)

    a, b = u1ml.Context(spec), u1ml.Context(spec)
    for c in (a, b):
        c.init_links(u1ml.HOT)
    a.sweeps(3)
    for k in range(3):
        sweep(b, 0, k)
    for e in range(len(ens)):
        assert np.array_equal(a.links(e), b.links(e))
        assert a.counter(e) == 3
        b.set_counter(3, e)
    a.multilevel()
    offset = 0
    outer = levels[0] if len(levels) == 2 else (0, 1, 0)
    for _ in range(outer[1]):
        for _ in range(outer[2]):
            sweep(b, outer[0], offset)
            offset += 1
        for _ in range(levels[-1][1] * levels[-1][2]):
            sweep(b, levels[-1][0], offset)
            offset += 1
    for e in range(len(ens)):
        assert np.array_equal(a.links(e), b.links(e))
        assert a.counter(e) == 3 + offset


# slices of 4, 32 and 108 links, enough of them that work-groups span slices
# (more waves than SIMDs, a tenth of their work-items idle slice by slice);
# 1100 slices are no whole number of work-groups
SHORT = [((2, 2, 2), 1100), ((4, 4, 4), 1100), ((6, 6, 6), 620)]


@pytest.mark.gpu
@pytest.mark.parametrize("ns,nt", SHORT)
def test_short_slices_match_oracle(ns, nt):
    """Work-groups over several time slices: overrelaxation of every direction
    and parity, all links and inside slabs of 2 and 4, with the bound of
    test_overrelaxation_matches_oracle."""
    import bench
    from oracle import oracle as O
    from paper_1309_3859_amd import u1ml

    V = int(np.prod(ns)) * nt
    spec = u1ml.Spec(ensembles=[u1ml.Ens(ns, nt, 1.1, seed=7, key_id=1)], levels=[(4, 1, 1), (2, 1, 1)], r=[1])
    ctx = u1ml.Context(spec)
    ref = O.Lattice(4, list(ns) + [nt], 1.1, seed=7, key_id=1)
    th0 = random_links(V, 5)
    size = bench.staple_abs(th0, ns, nt).reshape(-1)
    for mu, p, tau in itertools.product(range(4), (0, 1), (0, 2, 4)):
        print("phase", ns, nt, mu, p, tau, flush=True)
        ctx.set_links(th0)
        ref.set_links(th0)
        ctx.phase(1, mu, p, tau)
        ref.phase(1, mu, p, tau)
        d = circ_dist(ctx.links(0), ref.links())
        assert (d * size).max() < 1e-13


@pytest.mark.gpu
@pytest.mark.parametrize("ns,nt", SHORT)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("update", [0, 1])
def test_short_slices_equal_sweeps_in_lds(ns, nt, precision, update):
    """One launch per phase over short slices against sweeps inside slabs in
    LDS, bit for bit: every work-group size, heatbath retries by wave and (with
    small work-groups in FP64) by work-group, Metropolis, a lattice of longer
    slices in the batch."""
    from paper_1309_3859_amd import u1ml

    print("short slices", ns, nt, precision, update, flush=True)
    ens = [u1ml.Ens(ns, nt, 1.05, seed=3, key_id=0), u1ml.Ens((6, 8, 10), 4, 0.9, seed=3, key_id=1)]
    spec = u1ml.Spec(ensembles=ens, levels=[(2, 1, 1)], r=[1], precision=precision, n_or=2, update=update,
                     metro_delta=0.7)
    a = u1ml.Context(spec)
    a.init_links(u1ml.HOT)
    a.multilevel()
    for block in (64, 256, 1024):
        b = u1ml.Context(spec)
        b.set_block(block)
        b.init_links(u1ml.HOT)
        for k in range(3):
            kind = (u1ml.METROPOLIS if update else u1ml.HEATBATH) if k == 0 else u1ml.OVERRELAX
            for mu, p in itertools.product(range(4), (0, 1)):
                b.phase(kind, mu, p, 2, 0)
        for e in range(2):
            assert np.array_equal(a.links(e), b.links(e)), (block, e)


# (precision, lattice, betas, work-group sizes): launches of at least 640 (FP64) or 4096 (FP32) work-groups of at most
# 512 finish the heatbath's pending links by work-group, those of 1024 always by wave; the last work-group of
# every slice is not full
BY_GROUP = [(0, (30, 32, 34), (0.0, 0.2, 1.0), (64, 256, 512)), (1, (64, 62, 66), (0.3, 4.0), (64, 256, 512)),
            (0, (64, 62, 66), (1.1, 6.0), (128, 512))]


@pytest.mark.gpu
@pytest.mark.parametrize("precision,ns,betas,blocks", BY_GROUP)
@pytest.mark.parametrize("start", [0, 1])
def test_heatbath_retries_by_work_group_change_no_bit(precision, ns, betas, blocks, start):
    """Heatbath phases of every direction and parity, retries dealt over the
    work-group against retries dealt over the wave, from a cold and a hot start
    (few and many pending links) and, with beta = 0, with none."""
    from paper_1309_3859_amd import u1ml

    ens = [u1ml.Ens(ns, 4, b, seed=5, key_id=k) for k, b in enumerate(betas)]
    spec = u1ml.Spec(ensembles=ens, levels=[(2, 1, 1)], r=[1], precision=precision)
    want = None
    for block in (1024,) + blocks:
        print("heatbath by work-group", precision, ns, block, start, flush=True)
        ctx = u1ml.Context(spec)
        ctx.set_block(block)
        ctx.init_links(start)
        for mu, p, tau in itertools.product(range(4), (0, 1), (0, 2)):
            ctx.phase(u1ml.HEATBATH, mu, p, tau, pass_offset=tau + mu)
        got = [ctx.links(e) for e in range(len(ens))]
        ctx.close()
        if want is None:
            want = got
        for a, b in zip(want, got):
            assert np.array_equal(a, b), block


@pytest.mark.gpu
@pytest.mark.parametrize("levels,n_or", [([(2, 2, 2)], 3), ([(4, 2, 1), (2, 2, 1)], 2)])
@pytest.mark.parametrize("precision", [0, 1])
def test_lanes_and_graphs_change_no_bit_outside_lds(levels, n_or, precision):
    """Batches whose sweeps inside slabs are launches of both parities (their
    slabs too large for LDS) and, in the last one, launches of one phase: one,
    two and three lanes, graphs or direct launches, work-groups of 64 or 256."""
    from paper_1309_3859_amd import u1ml

    batches = [[((24, 24, 24), 4), ((12, 14, 16), 8), ((20, 10, 22), 4)],
               [((48, 48, 48), 8), ((32, 40, 36), 4), ((30, 20, 26), 8)]]
    for lattices in batches:
        ens = [u1ml.Ens(ns, nt, 1.0 - 0.02 * k, seed=9, key_id=k) for k, (ns, nt) in enumerate(lattices)]
        spec = u1ml.Spec(ensembles=ens, levels=levels, r=[1, 2], precision=precision, n_or=n_or, max_configs=2)
        want = None
        for lanes, graphs, block in ((1, True, 256), (2, True, 64), (3, False, 256), (2, False, 256)):
            print("lanes outside LDS", levels, precision, lattices[0], lanes, graphs, block, flush=True)
            ctx = u1ml.Context(spec)
            ctx.set_lanes(lanes)
            ctx.set_graphs(graphs)
            ctx.set_block(block)
            ctx.init_links(u1ml.HOT)
            ctx.sweeps(2)
            ctx.multilevel()
            ctx.multilevel()
            got = [ctx.results()] + [ctx.links(e) for e in range(3)] + [np.array([ctx.counter(e) for e in range(3)])]
            ctx.close()
            if want is None:
                want = got
            for a, b in zip(want, got):
                assert np.array_equal(a, b), (lanes, graphs, block)
