"""How many iterations a batched solve launches between its looks at the chains
must not show in the results: every chain bitwise as alone, also with a zero
right-hand side among the others, with starting guesses, and where cg_maxiter
cuts the solves off."""
import numpy as np
import pytest
import torch

from paper_0910_2950_amd import synth
from paper_0910_2950_amd.fgi import Action, Context

pytestmark = pytest.mark.gpu

MIX = [((4, 4, 4, 4), 5.6, 0.150), ((2, 2, 2, 2), 6.0, 0.157), ((6, 4, 4, 6), 5.8, 0.153)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("cg_batch", [1, 5, 16])
@pytest.mark.parametrize("prec,recon,maxiter,guess", [("fp64", 18, 2000, 0), ("mp32", 12, 2000, 1), ("mp16", 12, 2000, 1),
                                                     ("mp16", 12, 23, 0), ("fp64", 18, 23, 0)])
def test_rounds(cg_batch, prec, recon, maxiter, guess):
    ctx = Context(0)
    try:
        ctx.set_option("cg_batch", cg_batch)
        ctx.set_option("fg_start", guess)
        starts = [synth.hot_start(d, synth.SEED_BASE + 4600 + k) for k, (d, _, _) in enumerate(MIX)]
        etas = [s[2] for s in starts]
        etas[1] = np.zeros_like(etas[1])
        kw = dict(cg_tol=1e-10, prec=prec, link_recon=recon, cg_maxiter=maxiter)
        batch = [dict(dims=d, beta=b, kappa=k, U=dev(s[0]), P=dev(s[1]), eta=dev(e))
                 for (d, b, k), s, e in zip(MIX, starts, etas)]
        dHb, _ = ctx.trajectory_batched(batch, Action(beta=0.0, **kw), "FG", 0.5, 2, allow_noconv=maxiter < 100)
        for ch, s, e, dH in zip(batch, starts, etas, dHb):
            U, P = dev(s[0]), dev(s[1])
            dHs, _ = ctx.trajectory(ch["dims"], Action(beta=ch["beta"], kappa=ch["kappa"], **kw), "FG", 0.5, 2, U, P,
                                    dev(e), allow_noconv=maxiter < 100)
            assert torch.equal(U, ch["U"]) and torch.equal(P, ch["P"]) and dH == dHs, ch["dims"]
    finally:
        ctx.close()
