"""Options that choose a default by themselves can be given back to it."""
import numpy as np
import pytest
import torch

from paper_0910_2950_amd import fgi, synth
from paper_0910_2950_amd.fgi import Action, Context

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("prec,drop", [("mp32", 0.01), ("mp16", 0.1)])
def test_ru_delta_zero_is_the_default_by_storage(prec, drop):
    dims = (6, 4, 4, 6)
    U0, _, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4800)
    act = Action(beta=5.6, kappa=0.155, cg_tol=1e-12, prec=prec, link_recon=12)
    ctx = Context(0)
    try:
        def solve():
            X, st = ctx.cg_solve(dims, act, dev(U0), dev(eta))
            return X, st["cg_iters"], st["reliable_updates"]
        first = solve()
        ctx.set_option("ru_delta", 0.5)
        other = solve()
        assert other[2] > first[2]
        ctx.set_option("ru_delta", 0)
        again = solve()
        ctx.set_option("ru_delta", drop)
        named = solve()
        for r in (again, named):
            assert torch.equal(r[0], first[0]) and r[1:] == first[1:]
        for bad in (-0.1, 1.0, float("nan")):
            with pytest.raises(fgi.FgiError) as e:
                ctx.set_option("ru_delta", bad)
            assert e.value.code == fgi.FGI_EINVAL
    finally:
        ctx.close()
