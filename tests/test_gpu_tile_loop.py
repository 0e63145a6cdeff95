"""The tiled CG loop (RP_LOOP_AUTO on medium systems) against the three-launch
iteration: its products and vector updates are the same, its dot products add
a tile's rows first, so iterates after a fixed budget agree to rounding (1e-11
relative in FP64, far above what a reordered sum of this length changes) and
solves meet the same residual.  Sizes: just past the small systems' limit,
tiles that end inside a rank, with a partial last one, ranks of unequal size,
more ranks than tiles, a mesh whose far couplings all leave the tile; randomly
numbered meshes, whose tiles are cut from an order of the loop's own: ranks
numbered apart, a chain (regions of one dimension) and cells without a
coupling, which no region reaches.  Rows of more entries than a tile's slices
hold keep three launches, bit for bit."""
import numpy as np
import pytest

import oracle
import synth
from helpers import oracle_system, share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_AUTO, RP_LOOP_THREE, RP_LOOP_TWO_MAX_ROWS

pytestmark = pytest.mark.gpu

CASES = {
    "smallest": lambda: synth.small((52429, 5, 1), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=1),
    "one_rank": lambda: synth.small((65, 64, 64), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=2),
    "unequal_ranks": lambda: synth.small((70, 65, 90), ("rcb", 7), kappa=(1e-2, 1.0), seed=3),
    "many_ranks": lambda: synth.small((72, 70, 68), ("blocks", 7, 7, 7), kappa=(1e-1, 1.0), seed=4),
    "large_tiles": lambda: synth.small((104, 100, 96), ("blocks", 2, 3, 2), kappa=(1e-2, 1.0), seed=5),
    "random": lambda: synth.small((68, 66, 64), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=8, scramble=True),
    "random_ranks": lambda: synth.small((90, 85, 88), ("rcb", 5), kappa=(1e-2, 1.0), seed=9, scramble=True),
    "random_thin": lambda: synth.small((26243, 5, 2), ("blocks", 3, 1, 1), kappa=(1e-1, 1.0), seed=10, scramble=True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_agrees_with_three_launches(name):
    w = CASES[name]()
    m, _, v64, *_ = oracle_system(w)
    plan = make_plan(w)
    assert plan.n_rows > RP_LOOP_TWO_MAX_ROWS
    update(plan, share_values(w))
    b = w.rhs()
    x0 = np.random.default_rng(7).uniform(-1, 1, plan.n_rows)
    for budget in (1, 2, 30):
        for start in (None, x0):
            res = [plan.solve(dev_tensor(b), x=None if start is None else dev_tensor(start), tol=1e-13,
                              max_iter=budget, fused_loop=fl, check=False) for fl in (RP_LOOP_AUTO, RP_LOOP_THREE)]
            xa, xt = res[0][0].cpu().numpy(), res[1][0].cpu().numpy()
            assert res[0][1]["iters"] == res[1][1]["iters"] == budget
            assert np.linalg.norm(xa - xt) <= 1e-11 * np.linalg.norm(xt), (name, budget)
    for precision in ("fp64", "mixed", "mixed_rr"):
        x, info = plan.solve(dev_tensor(b), tol=1e-8, precision=precision)
        again, _ = plan.solve(dev_tensor(b), tol=1e-8, precision=precision)
        assert torch_mod().equal(x, again), "not deterministic"
        rr = oracle.true_relres(m, v64, b, x.cpu().numpy())
        assert info["status"] == 0 and info["restarts"] == 0 and rr <= 1e-8, (precision, info, rr)
    plan.close()


def test_values_follow_updates():
    w = synth.small((70, 66, 64), ("blocks", 2, 2, 2), kappa=(1e-1, 1.0), seed=6, timesteps=2)
    plan = make_plan(w)
    b = dev_tensor(w.rhs())
    for t in (0, 1):
        update(plan, share_values(w, t))
        for precision in ("fp64", "mixed"):
            x, info = plan.solve(b, tol=1e-8, precision=precision)
            xt, it = plan.solve(b, tol=1e-8, precision=precision, fused_loop=RP_LOOP_THREE)
            assert info["status"] == it["status"] == 0
            assert float((x - xt).norm()) <= 1e-6 * float(xt.norm()), (t, precision)
    plan.close()


def test_random_chain_with_uncoupled_cells():
    """A chain of 200 000 randomly numbered cells and 70 000 cells without a
    face: the seeds grow along the chain only, the cells alone fill regions by
    index."""
    n, c = 270000, 200000
    g = np.random.default_rng(11)
    chain = g.permutation(n)[:c].astype(np.int32)
    own, nbr = np.minimum(chain[:-1], chain[1:]), np.maximum(chain[:-1], chain[1:])
    o = np.lexsort((nbr, own))
    ranks = [dict(owner=own[o], neighbour=nbr[o], iface_cell=np.zeros(0, np.int32),
                  iface_nbr_rank=np.zeros(0, np.int32), iface_nbr_cell=np.zeros(0, np.int32))]
    from paper_2510_08536_amd import Plan
    plan = Plan([n], 0, 1, ranks)
    plan.update([np.full(n, 2.5)], [np.full(c - 1, -1.0)], [np.zeros(0)])
    b = dev_tensor(g.uniform(-1, 1, n))
    for precision, bar in (("fp64", 1e-11), ("mixed", 1e-9)):
        xa, ia = plan.solve(b, tol=1e-10, precision=precision)
        xt, it = plan.solve(b, tol=1e-10, precision=precision, fused_loop=RP_LOOP_THREE)
        assert ia["status"] == it["status"] == 0 and ia["iters"] == it["iters"]
        assert float((xa - xt).norm()) <= bar * float(xt.norm()), precision
    plan.close()


def test_long_rows_keep_three_launches():
    w = synth.small((68, 66, 64), ("blocks", 2, 1, 1), kappa=(1e-1, 1.0), seed=12, stencil=27)
    plan = make_plan(w)
    update(plan, share_values(w))
    b = dev_tensor(w.rhs())
    res = [plan.solve(b, tol=1e-8, fused_loop=fl) for fl in (RP_LOOP_AUTO, RP_LOOP_THREE)]
    assert torch_mod().equal(res[0][0], res[1][0]) and res[0][1] == res[1][1]
    plan.close()
