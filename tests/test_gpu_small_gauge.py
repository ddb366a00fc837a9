"""The small-lattice forms of the gauge force (a link's six staples shared by six
waves) and of the link update (the exponential's series), against the oracle.

The force sums 12 products of unit-size numbers per entry: 1e-13 relative as for
every force kernel; the improved staples 24 products more (c1 = 0.3: the rectangles
the larger part).  The series is exact to a few eps for norms up to 1 and hands
larger ones to the closed form; both sides of that line are drawn, and the edge
of the sizes that take it (2048 sites) from both sides: 2e-14 as for the
exponential, one more product for the link."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_0910_2950_amd import fgi, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = fgi.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 2, 4), (6, 4, 4, 6), (8, 8, 8, 16), (8, 8, 8, 18)])
def test_force(ctx, dims):
    U0, _, _, _ = synth.hot_start(dims, synth.SEED_BASE + 4400, fermions=False)
    F = ctx.gauge_force(dims, 5.7, dev(U0)).cpu().numpy()
    ref = orc.gauge_force(dims, 5.7, U0)
    assert np.max(np.abs(F - ref)) <= 1e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 2, 4), (6, 4, 4, 6), (8, 8, 8, 16), (8, 8, 8, 18)])
@pytest.mark.parametrize("c1", [-1.0 / 12.0, 0.3])
def test_improved_force(ctx, dims, c1):
    U0, _, _, _ = synth.hot_start(dims, synth.SEED_BASE + 4400, fermions=False)
    F, _ = ctx.force(dims, fgi.Action(beta=5.7, c1=c1), dev(U0))
    F = F.cpu().numpy()
    ref = orc.gauge_force(dims, 5.7, U0, c1=c1)
    assert np.max(np.abs(F - ref)) <= 1e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 4, 6), (8, 8, 8, 4), (8, 8, 8, 6)])
@pytest.mark.parametrize("h", [0.0, 1e-9, 1e-4, 0.1, 0.4, 0.6, 2.5])
def test_link_update(ctx, dims, h):
    U0, P0, _, _ = synth.hot_start(dims, synth.SEED_BASE + 4500, fermions=False)
    U = ctx.link_update(dims, h, dev(P0), dev(U0)).cpu().numpy()
    assert np.max(np.abs(U - orc.link_update(dims, h, P0, U0))) <= 2.5e-14


@pytest.mark.parametrize("c1", [0.0, -1.0 / 12.0])
@pytest.mark.parametrize("sizes", [[(4, 4, 4, 4)] * 32, [(4, 4, 4, 4)] * 33, [(2, 2, 2, 2), (8, 8, 8, 16), (8, 8, 8, 18)],
                                   [(6, 6, 6, 6)] * 3 + [(8, 8, 8, 8)], [(6, 6, 6, 6)] * 38])
def test_batch_equals_single_runs_whatever_its_volume(ctx, sizes, c1):
    """A batch's total volume chooses between the force kernels (8192 sites, 49152
    for ragged chains, from both sides and mixed): bitwise the chains' own runs."""
    starts = {}
    for d in sizes:
        if d not in starts:
            starts[d] = [synth.hot_start(d, synth.SEED_BASE + 4450 + k, fermions=False)[:2] for k in range(2)]
    chains, single = [], []
    for k, d in enumerate(sizes):
        U0, P0 = starts[d][k % 2]
        U, P = dev(U0), dev(P0)
        dH, _ = ctx.trajectory(d, fgi.Action(beta=5.5 + 0.01 * k, c1=c1), "FG", 0.25, 2, U, P)
        single.append((U, P, dH))
        chains.append(dict(dims=d, beta=5.5 + 0.01 * k, kappa=0.0, U=dev(U0), P=dev(P0)))
    dH, _ = ctx.trajectory_batched(chains, fgi.Action(beta=0.0, c1=c1), "FG", 0.25, 2)
    for ch, d, (U, P, d1) in zip(chains, dH, single):
        assert torch.equal(ch["U"], U) and torch.equal(ch["P"], P) and d == d1, ch["dims"]
