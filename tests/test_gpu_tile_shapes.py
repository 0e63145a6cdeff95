"""The tiled loops at every number of rows per thread they are built for, which
smaller meshes do not reach: FP64 CG from 9 to 16, FP32 from 18 to 32, BiCGStab
from 5 to 10 (the places are then read anew every iteration, and x stays in
memory).  Against the launched kernels after a fixed budget: 1e-11 relative in
FP64 (1e-10 for BiCGStab), 1e-4 for FP32 iterations (rounding of reordered sums
of some 300 terms of a thread and a tree over 4 million rows).  A whole solve
meets its residual, formed by the library's own product, and is not the launched
one's to the bit, which it would be on launched kernels.  (One iteration may be:
its one scalar can round alike.)"""
import pytest

import synth
from helpers import share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_THREE

pytestmark = pytest.mark.gpu

ROWS = 256 * 512   # rows of 256 tiles with a row per thread


def _mesh(rows_per_thread, **kw):
    return synth.small((50, 50, ROWS * rows_per_thread // 2500), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=91, **kw)


def _compare(plan, b, budgets, bar, **kw):
    torch = torch_mod()
    for budget in budgets:
        x, info = plan.solve(b, tol=1e-13, max_iter=budget, check=False, **kw)
        x3, info3 = plan.solve(b, tol=1e-13, max_iter=budget, check=False, fused_loop=RP_LOOP_THREE, **kw)
        assert info["iters"] == info3["iters"] == budget
        assert float((x - x3).norm()) <= bar * float(x3.norm()), budget
    x, info = plan.solve(b, tol=1e-8, **kw)
    x3, info3 = plan.solve(b, tol=1e-8, fused_loop=RP_LOOP_THREE, **kw)
    assert info["status"] == info3["status"] == 0 and info["rel_res"] <= 1e-8
    assert not torch.equal(x, x3), "launched kernels"
    if not kw.get("transpose"):
        assert float((b - plan.spmv(x)).norm()) <= 1e-8 * (1 + 1e-6) * float(b.norm())


@pytest.mark.parametrize("rows", [9, 10, 11, 12, 13, 14, 15, 16])
def test_cg_fp64(rows):
    w = _mesh(rows)
    plan = make_plan(w)
    update(plan, share_values(w))
    _compare(plan, dev_tensor(w.rhs()), (1, 2, 30), 1e-11)
    plan.close()


@pytest.mark.parametrize("rows", [18, 20, 22, 24, 28, 32])
def test_cg_fp32(rows):
    w = _mesh(rows)
    plan = make_plan(w)
    update(plan, share_values(w))
    _compare(plan, dev_tensor(w.rhs()), (1, 2), 1e-4, precision="mixed")
    plan.close()


@pytest.mark.parametrize("rows", [5, 6, 7, 8, 9, 10])
def test_bicgstab(rows):
    w = _mesh(rows)
    plan = make_plan(w)
    update(plan, share_values(w, values=w.momentum_values(pe=3.0)), lower=True)
    b = dev_tensor(w.rhs())
    _compare(plan, b, (1, 2), 1e-10, method="bicgstab")
    _compare(plan, b, (1, 2), 1e-10, method="bicgstab", transpose=1)
    plan.close()


def test_an_order_of_the_loop_follows_updates():
    """Randomly numbered cells, whose tiles are cut from a row order: one plan,
    new values, A and A^T in turn."""
    w = synth.small((68, 66, 64), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=92, scramble=True, timesteps=3)
    plan = make_plan(w)
    b = dev_tensor(w.rhs())
    for t in (0, 1, 2, 0):
        update(plan, share_values(w, t))
        _compare(plan, b, (1, 10), 1e-11)
        _compare(plan, b, (1, 2), 1e-4, precision="mixed")
        update(plan, share_values(w, values=w.momentum_values(t)), lower=True)
        _compare(plan, b, (1, 2), 1e-10, method="bicgstab", transpose=1)
        _compare(plan, b, (1, 2), 1e-10, method="bicgstab")
    plan.close()
