"""Where cg_maxiter cuts a solve off: the limit itself may be as large as an int
holds."""
import numpy as np
import pytest
import torch

from paper_0910_2950_amd import synth
from paper_0910_2950_amd.fgi import Action, Context

pytestmark = pytest.mark.gpu
DIMS = (4, 4, 4, 4)


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("prec,recon,csw", [("fp64", 18, 0.0), ("mp32", 18, 0.0), ("mp16", 12, 0.0), ("mp32", 18, 1.0)])
def test_largest_limit(ctx, prec, recon, csw):
    """cg_maxiter = 2^31 - 1 gives the bits and counts of any limit that is not reached."""
    U0, _, eta, _ = synth.hot_start(DIMS, synth.SEED_BASE + 4700)
    out = []
    for maxiter in (20000, 2**31 - 8, 2**31 - 1):
        act = Action(beta=5.6, kappa=0.15, cg_tol=1e-11, cg_maxiter=maxiter, prec=prec, link_recon=recon, csw=csw)
        out.append(ctx.cg_solve(DIMS, act, dev(U0), dev(eta)))
    for X, st in out[1:]:
        assert torch.equal(X, out[0][0]) and st["cg_iters"] == out[0][1]["cg_iters"] > 0
        assert st["max_rel_resid"] == out[0][1]["max_rel_resid"] <= 1e-11
