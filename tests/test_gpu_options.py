"""Options that choose a default by themselves can be given back to it, and the
autotuner leaves alone what it cannot measure."""
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


@pytest.mark.parametrize("block", [64, 128, 256])
def test_autotuner_leaves_the_block_size_of_split_lattices(block):
    """On lattices whose Dslash-shaped kernels have their own block size, the option
    stays the caller's (it rules larger lattices of the same context)."""
    dims = (8, 8, 8, 8)
    U0, P0, eta, _ = synth.hot_start(dims, synth.SEED_BASE + 4810)
    U, P, e = dev(U0), dev(P0), dev(eta)
    ctx = Context(0)
    try:
        ctx.set_option("dslash_block", block)
        act = Action(beta=5.6, kappa=0.155, cg_tol=1e-10, prec="mp16", link_recon=12)
        t = ctx.autotune_cg(dims, act, U, e)
        tb = ctx.autotune_batched([dict(dims=dims, beta=5.6, kappa=0.155, U=U, P=P, eta=e)] * 2, act)
        for r in (t, tb):
            s = r["sched_us_per_iter"]
            assert r["dslash_block"] == block and s[0] == s[2] == s[4] > 0 and s[1] == s[3] == s[5] > 0
            assert s[r["xcd_order"]] == min(s)
        # fixed-point links keep one thread per site: every block size is timed
        r = ctx.autotune_cg(dims, Action(beta=5.6, kappa=0.155, cg_tol=1e-10, prec="mp16"), U, e)
        s = r["sched_us_per_iter"]
        assert len(set(s)) > 2 and s[2 * [64, 128, 256].index(r["dslash_block"]) + r["xcd_order"]] == min(s)
    finally:
        ctx.close()
