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
