"""The two ways between the user's layout and the checkerboard planes, on both sides
of the volumes that choose between them (links 16384 sites, 32768 inwards where a
plane is a multiple of 2048; momenta 65536 inwards, 4096 outwards), with last blocks
partly filled: exact, and a call's inputs (links with momenta, links with a spinor) in
one launch as one by one."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_0910_2950_amd import synth
from paper_0910_2950_amd.fgi import Action, Context

pytestmark = pytest.mark.gpu
DIMS = [(8, 8, 8, 8), (6, 10, 14, 6), (8, 8, 16, 16), (10, 10, 14, 12), (16, 16, 16, 8), (10, 14, 16, 18),
        (16, 16, 16, 16), (10, 14, 22, 22)]


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


def planes(dims, a):
    """[4, V, n] -> [4, parity, n, Vh]"""
    x = [np.arange(d) for d in dims]
    par = (x[0][None, None, None, :] + x[1][None, None, :, None] + x[2][None, :, None, None] + x[3][:, None, None, None]) & 1
    par = par.reshape(-1)
    return np.stack([a[:, par == p].transpose(0, 2, 1) for p in (0, 1)], 1)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("kind,dtype,shape", [("links", np.complex128, (3, 3)), ("momenta", np.float64, (8,))])
def test_round_trip(ctx, dims, kind, dtype, shape):
    v, n = int(np.prod(dims)), int(np.prod(shape))
    rng = np.random.default_rng(6)
    a = rng.standard_normal((4, v, n)).astype(dtype)
    if dtype is np.complex128:
        a = a + 1j * rng.standard_normal((4, v, n))
    t = torch.from_numpy(a.reshape((4, v) + shape)).cuda()
    buf = ctx.field_pack(dims, kind, t)
    got = buf.cpu().numpy().view(dtype)[: a.size].reshape(4, 2, n, v // 2)
    assert np.array_equal(got, planes(dims, a))
    assert torch.equal(ctx.field_unpack(dims, kind, buf), t)


@pytest.mark.parametrize("dims", [(8, 8, 16, 16), (10, 10, 14, 12)])
def test_inputs_in_one_launch(ctx, dims):
    """2e-14 as for the exponential, 1e-14 for two hops"""
    U0, P0, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4950)
    U, P, e = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (U0, P0, eta))
    out = ctx.link_update(dims, 0.1, P, U.clone()).cpu().numpy()
    assert np.max(np.abs(out - orc.link_update(dims, 0.1, P0, U0))) <= 2.5e-14
    out = ctx.mhat(dims, Action(beta=5.6, kappa=0.14), U, e).cpu().numpy()
    ref = orc.mhat(dims, 0.14, U0, eta)
    assert np.max(np.abs(out - ref)) <= 1e-14 * np.max(np.abs(ref))
