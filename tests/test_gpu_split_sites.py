"""The Dslash-shaped kernels that share a site between four waves (lattices of
at most 32768 even sites) against the oracle, at the sizes where they can go
wrong: fewer sites than a block of 64 holds, a partly filled last block, and
both sides of the line to the one-thread-per-site kernels.

Tolerances: a hop sums 24 products of unit-size numbers and is applied twice,
so 1e-14 relative to the largest component (eps ~ 1e-16 times a few tens); a CG
solution stops at 1e-13 and the smallest eigenvalue of Mhat^+ Mhat on these
fields is above 1e-2, so 1e-10 in FP64 and, with the same FP64 true residual
deciding, in mixed precision."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_0910_2950_amd import fgi, synth

pytestmark = pytest.mark.gpu
DIMS = [(2, 2, 2, 2), (4, 4, 2, 4), (4, 4, 4, 4), (6, 4, 4, 6), (2, 14, 6, 10), (16, 16, 16, 16), (16, 16, 16, 18)]


@pytest.fixture(scope="module")
def ctx():
    c = fgi.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("dagger", [False, True])
def test_mhat(ctx, dims, dagger):
    U0, _, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4100)
    out = ctx.mhat(dims, fgi.Action(beta=5.6, kappa=0.15), dev(U0), dev(eta), dagger=dagger).cpu().numpy()
    ref = orc.mhat(dims, 0.15, U0, eta, dagger=dagger)
    assert np.max(np.abs(out - ref)) <= 1e-14 * np.max(np.abs(ref))


@pytest.mark.parametrize("dims", DIMS[1:])
@pytest.mark.parametrize("prec,recon", [("fp64", 18), ("mp32", 18), ("mp32", 12), ("mp16", 18), ("mp16", 12)])
@pytest.mark.parametrize("form", [0, 1])
def test_solve(ctx, dims, prec, recon, form):
    U0, _, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4200)
    ctx.set_option("cg_form", form)
    try:
        X, st = ctx.cg_solve(dims, fgi.Action(beta=5.6, kappa=0.15, cg_tol=1e-13, prec=prec, link_recon=recon), dev(U0),
                             dev(eta))
    finally:
        ctx.set_option("cg_form", 0)
    assert st["status"] == 0 and st["max_rel_resid"] <= 1e-13
    X = X.cpu().numpy()
    r = eta - orc.mhat(dims, 0.15, U0, orc.mhat(dims, 0.15, U0, X), dagger=True)
    assert np.linalg.norm(r) <= 1.1e-13 * np.linalg.norm(eta)
    ref = orc.cg(dims, 0.15, U0, eta, tol=1e-14)[0]
    assert np.max(np.abs(X - ref)) <= 1e-10 * np.max(np.abs(ref))


def test_batch_of_both_kinds_equals_single_runs(ctx):
    """Chains on both sides of the line in one batch: bitwise their own runs."""
    act = fgi.Action(beta=5.6, kappa=0.15, cg_tol=1e-10, prec="mp16", link_recon=12)
    chains, single = [], []
    for k, dims in enumerate([(4, 4, 4, 4), (16, 16, 16, 18), (6, 4, 4, 6)]):
        U0, P0, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4300 + k)
        U, P = dev(U0), dev(P0)
        a = fgi.Action(beta=5.5 + 0.1 * k, kappa=0.15, cg_tol=1e-10, prec="mp16", link_recon=12)
        dH, _ = ctx.trajectory(dims, a, "FG", 0.25, 1, U, P, dev(eta))
        single.append((U, P, dH))
        chains.append(dict(dims=dims, beta=a.beta, kappa=0.15, U=dev(U0), P=dev(P0), eta=dev(eta)))
    dH, _ = ctx.trajectory_batched(chains, act, "FG", 0.25, 1)
    for ch, d, (U, P, d1) in zip(chains, dH, single):
        assert torch.equal(ch["U"], U) and torch.equal(ch["P"], P) and d == d1
