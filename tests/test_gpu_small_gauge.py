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
