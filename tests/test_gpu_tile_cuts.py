"""Systems whose ranks do not divide into tiles evenly: cut by rank they take
more rows per thread than a loop has registers for, cut in one run they do not.
The tiled loop is taken: iterates after a fixed budget agree with the launched
kernels' to 1e-11 relative in FP64 (1e-10 for BiCGStab, reordered sums) and are
not the same bits, which they are where both take the launched kernels."""
import pytest

import synth
from helpers import share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_THREE

pytestmark = pytest.mark.gpu

# 18 and 20 rows per thread by rank, 16 in one run (CG's limit in FP64); 11 against 10 (BiCGStab's)
CASES = [("cg", 128, (3, 3, 3)), ("cg", 128, (3, 3, 5)), ("bicgstab", 108, (3, 3, 3)), ("bicgstab", 108, (4, 4, 3))]


@pytest.mark.parametrize("method,side,ranks", CASES)
def test_the_loop_is_taken(method, side, ranks):
    w = synth.small((side, side, side), ("blocks", *ranks), kappa=(1e-1, 1.0), seed=61)
    plan = make_plan(w)
    bi = method == "bicgstab"
    update(plan, share_values(w, values=w.momentum_values(pe=3.0)) if bi else share_values(w), lower=bi)
    b = dev_tensor(w.rhs())
    kw = dict(tol=1e-13, max_iter=2 if bi else 10, method=method, check=False)
    x, info = plan.solve(b, **kw)
    x3, info3 = plan.solve(b, fused_loop=RP_LOOP_THREE, **kw)
    assert info["iters"] == info3["iters"] == kw["max_iter"]
    assert float((x - x3).norm()) <= (1e-10 if bi else 1e-11) * float(x3.norm())
    assert not torch_mod().equal(x, x3), "launched kernels"
    plan.close()
