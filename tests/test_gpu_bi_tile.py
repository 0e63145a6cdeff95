"""The one-launch BiCGStab loop (RP_LOOP_AUTO where the system fits it)
against the launched kernels (RP_LOOP_THREE), which sum the dot products in
another order: iterates after one and two iterations agree to 1e-10 relative
(rounding of the sums, some 1e-15, times the growth of two iterations), solves
meet the same residual, the transposed system included.  Sizes: one row per
thread and less, tiles that end inside a rank, the first size with two rows per
thread, randomly numbered cells, more rows per thread than x has registers
for.  Long rows keep the launched kernels, bit for bit."""
import numpy as np
import pytest

import oracle
import synth
from helpers import share_ranks, share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_ERR_BREAKDOWN, RP_LOOP_AUTO, RP_LOOP_THREE

pytestmark = pytest.mark.gpu

CASES = {
    "tiny": lambda: synth.small((3, 2, 1), ("blocks", 1, 1, 1), seed=1),
    "one_tile": lambda: synth.small((8, 8, 8), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=2),
    "one_row_more": lambda: synth.small((27, 19, 1), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=3),
    "ragged_ranks": lambda: synth.small((40, 33, 29), ("rcb", 7), kappa=(1e-1, 1.0), seed=4),
    "two_rows": lambda: synth.small((51, 52, 50), ("blocks", 2, 1, 2), kappa=(1e-1, 1.0), seed=5),
    "random": lambda: synth.small((70, 66, 64), ("rcb", 3), kappa=(1e-1, 1.0), seed=6, scramble=True),
    "x_in_memory": lambda: synth.small((98, 95, 96), ("blocks", 2, 2, 2), kappa=(1e-1, 1.0), seed=7),
}


def _setup(w):
    v = w.momentum_values(pe=3.0)
    m = oracle.merge(w.part.n_cells, 0, w.n_ranks, share_ranks(w))
    vals = share_values(w, values=v)
    val64, *_ = oracle.update(m, oracle.receive_buffer(vals))
    plan = make_plan(w)
    update(plan, vals, lower=True)
    return m, val64, plan


@pytest.mark.parametrize("name", sorted(CASES))
def test_agrees_with_launched_kernels(name):
    import scipy.sparse as sp
    w = CASES[name]()
    m, val64, plan = _setup(w)
    A = sp.csr_matrix((val64, m.col, m.row_ptr), shape=(m.n_rows, m.n_rows))
    b = w.rhs()
    x0 = np.random.default_rng(7).uniform(-1, 1, plan.n_rows)
    for transpose in (0, 1):
        for budget in (1, 2):
            for start in (None, x0):
                res = [plan.solve(dev_tensor(b), x=None if start is None else dev_tensor(start), tol=1e-13,
                                  method="bicgstab", transpose=transpose, max_iter=budget, fused_loop=fl, check=False)
                       for fl in (RP_LOOP_AUTO, RP_LOOP_THREE)]
                xa, xt = res[0][0].cpu().numpy(), res[1][0].cpu().numpy()
                assert res[0][1]["iters"] == res[1][1]["iters"]
                assert np.linalg.norm(xa - xt) <= 1e-10 * np.linalg.norm(xt), (name, transpose, budget)
        kw = dict(tol=1e-9, method="bicgstab", transpose=transpose)
        x, info = plan.solve(dev_tensor(b), **kw)
        again, _ = plan.solve(dev_tensor(b), **kw)
        assert torch_mod().equal(x, again), "not deterministic"
        xh = x.cpu().numpy()
        rr = np.linalg.norm(b - (A.T if transpose else A) @ xh) / np.linalg.norm(b)
        assert info["status"] == 0 and rr <= 1e-9 * (1 + 1e-6), (transpose, info, rr)
    plan.close()


def test_values_follow_updates_and_transposes():
    """One plan, solves of A, A^T and A of new values in turn, CG between."""
    w = synth.small((66, 65, 64), ("blocks", 2, 2, 1), kappa=(1e-1, 1.0), seed=8, timesteps=2)
    plan = make_plan(w)
    b = dev_tensor(w.rhs())
    for t in (0, 1):
        update(plan, share_values(w, values=w.momentum_values(t)), lower=True)
        for transpose in (0, 1, 0):
            res = [plan.solve(b, tol=1e-10, method="bicgstab", transpose=transpose, fused_loop=fl)
                   for fl in (RP_LOOP_AUTO, RP_LOOP_THREE)]
            assert all(i["status"] == 0 for _, i in res)
            assert float((res[0][0] - res[1][0]).norm()) <= 1e-7 * float(res[1][0].norm()), (t, transpose)
        update(plan, share_values(w, t))
        res = [plan.solve(b, tol=1e-9, fused_loop=fl)[0] for fl in (RP_LOOP_AUTO, RP_LOOP_THREE)]
        assert float((res[0] - res[1]).norm()) <= 1e-6 * float(res[1].norm()), t
    plan.close()


def test_breakdown_and_long_rows():
    """(r^, A M^-1 r^) = 0 at once on [[1, -1], [-1, 1]] with b = (1, 1): both
    loops report it at iteration 0.  27-point rows do not fit a tile's slices."""
    from paper_2510_08536_amd import Plan
    ranks = [dict(owner=np.array([0], np.int32), neighbour=np.array([1], np.int32), iface_cell=np.zeros(0, np.int32),
                  iface_nbr_rank=np.zeros(0, np.int32), iface_nbr_cell=np.zeros(0, np.int32))]
    plan = Plan([2], 0, 1, ranks)
    plan.update([np.array([1.0, 1.0])], [np.array([-1.0])], [np.zeros(0)], lower=[np.array([-1.0])])
    for fl in (RP_LOOP_AUTO, RP_LOOP_THREE):
        _, info = plan.solve(dev_tensor(np.array([1.0, 1.0])), method="bicgstab", fused_loop=fl, check=False)
        assert info["status"] == RP_ERR_BREAKDOWN and info["iters"] == 0, (fl, info)
    plan.close()
    w = synth.small((20, 19, 18), ("blocks", 2, 1, 1), kappa=(1e-1, 1.0), seed=9, stencil=27)
    plan = make_plan(w)
    update(plan, share_values(w))
    res = [plan.solve(dev_tensor(w.rhs()), tol=1e-9, method="bicgstab", fused_loop=fl)
           for fl in (RP_LOOP_AUTO, RP_LOOP_THREE)]
    assert torch_mod().equal(res[0][0], res[1][0]) and res[0][1] == res[1][1]
    plan.close()
