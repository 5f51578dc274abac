"""Slab products and their sums over the lattice, one measurement of given
links without updates: C(r) is then the plain Polyakov-loop correlator, formed
here with numpy.  The lattices take one, two, a partial third and, for the
waves that add the work-groups' partial sums 64 at a time, more than 64
work-groups of 1024 sites a separation."""
import numpy as np
import pytest

from helpers.inputs import random_links

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nt", [((4, 4, 4), 4), ((16, 16, 8), 4), ((26, 10, 8), 6), ((48, 48, 32), 4)])
def test_correlators_of_given_links(ns, nt):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1309_3859_amd import u1ml

    vol = ns[0] * ns[1] * ns[2] * nt
    th = random_links(vol, 29)
    seps = [1, 2, ns[0] // 2]
    spec = u1ml.Spec(ensembles=[u1ml.Ens(ns, nt, 1.0, seed=1)], levels=[(2, 1, 0)], r=seps, dirs=[0],
                     precision=u1ml.FP64, max_configs=1)
    ctx = u1ml.Context(spec)
    ctx.set_links(th, 0)
    ctx.multilevel()
    got = spec.unpack(ctx.results()[0, 0])["C"]
    a = th.reshape(nt, ns[2], ns[1], ns[0], 4)[..., 3].sum(axis=0)
    p = np.exp(1j * a)
    want = np.array([np.mean(np.conj(p) * np.roll(p, -r, axis=2)) for r in seps])
    # |p| = 1; each angle sum of Nt terms below Nt pi rounds by at most Nt (Nt pi) 2^-53 on either side, at both
    # ends, and each of the Nt / 2 slab factors by two units in the last place
    bound = 4 * nt * nt * np.pi * 2.0**-53 + 2 * nt * 2.0**-52
    print(ns, nt, np.abs(got - want).max(), bound, flush=True)
    assert np.abs(got - want).max() <= bound
