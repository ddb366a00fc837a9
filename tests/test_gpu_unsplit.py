"""The Dslash-shaped kernels with one thread per site, in every block size, where
lattices or links take them: above 32768 even sites, and with 16-bit fixed-point
links on any lattice.  40040 even sites leave a last block partly filled in every
size, and so do the chains of the batch.

Tolerances: a solve stops at a true residual of tol, which the oracle's operator
confirms to 10 %; a site's hops are summed in the same order by the kernels that
share a site between waves and by these, so on a lattice repeated in x both give the
same bits in FP64 and FP32 (in FP16 the compiler fuses the scaling of the stored
numbers into the projection differently in the two)."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_0910_2950_amd import synth
from paper_0910_2950_amd.fgi import Action, Context

pytestmark = pytest.mark.gpu
LARGE = (10, 14, 22, 26)
BLOCKS = [(64, 1), (128, 0), (256, 1)]


@pytest.fixture
def ctx():
    c = Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def large():
    U0, _, eta, _ = synth.hot_start(LARGE, synth.SEED_BASE + 4900)
    return U0, eta, dev(U0), dev(eta)


def schedule(ctx, block, order):
    ctx.set_option("dslash_block", block)
    ctx.set_option("xcd_order", order)


@pytest.mark.parametrize("block,order", BLOCKS)
@pytest.mark.parametrize("csw", [0.0, 1.0])
def test_operator(ctx, large, block, order, csw):
    U0, eta, U, e = large
    schedule(ctx, block, order)
    for dagger in (False, True):
        out = ctx.mhat(LARGE, Action(beta=5.6, kappa=0.14, csw=csw), U, e, dagger=dagger).cpu().numpy()
        ref = orc.clover_mhat(LARGE, 0.14, csw, U0, eta, dagger=dagger) if csw else orc.mhat(LARGE, 0.14, U0, eta,
                                                                                             dagger=dagger)
        assert np.max(np.abs(out - ref)) <= (1e-13 if csw else 1e-14) * np.max(np.abs(ref))


@pytest.mark.parametrize("block,order", BLOCKS)
@pytest.mark.parametrize("prec,recon,csw,form", [("fp64", 18, 0.0, 0), ("mp32", 18, 0.0, 0), ("mp16", 12, 0.0, 0),
                                                 ("mp16", 12, 0.0, 1), ("fp64", 18, 1.0, 0), ("mp32", 18, 1.0, 0),
                                                 ("mp32", 12, 1.0, 0)])
def test_solve(ctx, large, block, order, prec, recon, csw, form):
    U0, eta, U, e = large
    schedule(ctx, block, order)
    ctx.set_option("cg_form", form)
    act = Action(beta=5.6, kappa=0.14, csw=csw, cg_tol=1e-11, prec=prec, link_recon=recon)
    X, st = ctx.cg_solve(LARGE, act, U, e)
    X2, _ = ctx.cg_solve(LARGE, act, U, e)
    assert torch.equal(X, X2) and st["max_rel_resid"] <= 1e-11
    X = X.cpu().numpy()
    if csw:
        r = eta - orc.clover_mhat(LARGE, 0.14, csw, U0, orc.clover_mhat(LARGE, 0.14, csw, U0, X), dagger=True)
    else:
        r = eta - orc.mhat(LARGE, 0.14, U0, orc.mhat(LARGE, 0.14, U0, X), dagger=True)
    assert np.linalg.norm(r) <= 1.1e-11 * np.linalg.norm(eta)


@pytest.mark.parametrize("block,order", BLOCKS)
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 4, 6)])
@pytest.mark.parametrize("form", [0, 1])
def test_fixed_point_links_on_small_lattices(ctx, block, order, dims, form):
    U0, _, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4910)
    schedule(ctx, block, order)
    ctx.set_option("cg_form", form)
    X, st = ctx.cg_solve(dims, Action(beta=5.6, kappa=0.14, cg_tol=1e-11, prec="mp16"), dev(U0), dev(eta))
    assert st["max_rel_resid"] <= 1e-11
    X = X.cpu().numpy()
    r = eta - orc.mhat(dims, 0.14, U0, orc.mhat(dims, 0.14, U0, X), dagger=True)
    assert np.linalg.norm(r) <= 1.1e-11 * np.linalg.norm(eta)


@pytest.mark.parametrize("block,order", BLOCKS)
def test_batch_of_fixed_point_links_equals_single_runs(ctx, block, order):
    schedule(ctx, block, order)
    kw = dict(cg_tol=1e-10, prec="mp16", link_recon=18)
    chains, single = [], []
    for k, dims in enumerate([(2, 2, 2, 2), (6, 4, 4, 6), (4, 4, 4, 4), (6, 6, 6, 6)]):
        U0, P0, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4920 + k)
        U, P = dev(U0), dev(P0)
        dH, _ = ctx.trajectory(dims, Action(beta=5.5 + 0.1 * k, kappa=0.15, **kw), "FG", 0.25, 1, U, P, dev(eta))
        single.append((U, P, dH))
        chains.append(dict(dims=dims, beta=5.5 + 0.1 * k, kappa=0.15, U=dev(U0), P=dev(P0), eta=dev(eta)))
    dH, _ = ctx.trajectory_batched(chains, Action(beta=0.0, **kw), "FG", 0.25, 1)
    for ch, d, (U, P, d1) in zip(chains, dH, single):
        assert torch.equal(ch["U"], U) and torch.equal(ch["P"], P) and d == d1, ch["dims"]


def twice_in_x(f, dims, half):
    """A field over (…, sites, …) repeated along x; half: even or odd sites only."""
    lead = f.shape[:1] if not half else ()
    lx = dims[0] // 2 if half else dims[0]
    g = f.reshape(*lead, -1, lx, *f.shape[len(lead) + 1:])
    return torch.cat([g, g], len(lead) + 1).reshape(*lead, -1, *f.shape[len(lead) + 1:]).contiguous()


@pytest.mark.parametrize("prec,recon", [("fp64", 18), ("mp32", 18), ("mp32", 12)])
def test_split_and_unsplit_hops_have_the_same_bits(ctx, prec, recon):
    dims, twice = (16, 16, 16, 16), (32, 16, 16, 16)
    U0, _, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4930)
    U, e = dev(U0), dev(eta)
    U2, e2 = twice_in_x(U, dims, False), twice_in_x(e, dims, True)
    act = Action(beta=5.6, kappa=0.14, prec=prec, link_recon=recon)
    for parity in (0, 1):
        a = ctx.dslash(dims, act, U, e, parity, prec=prec)
        b = ctx.dslash(twice, act, U2, e2, parity, prec=prec)
        assert torch.equal(twice_in_x(a, dims, True), b)
    if prec == "fp64":
        for csw in (0.0, 1.0):
            act = Action(beta=5.6, kappa=0.14, csw=csw)
            for dagger in (False, True):
                a = ctx.mhat(dims, act, U, e, dagger=dagger)
                b = ctx.mhat(twice, act, U2, e2, dagger=dagger)
                diff = float((twice_in_x(a, dims, True) - b).abs().max())
                assert diff == 0.0 if csw == 0.0 else diff <= 1e-14
