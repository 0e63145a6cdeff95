"""The one-launch loops where memory runs out, the device's or (while the tiles
are built) the host's: any of the allocations they ask for fails, alone or with
all that follow.  A solve then takes the tiles that are left to it or the
launched kernels, and so does every later one, whatever memory there is by
then: iterates after a fixed budget agree with RP_LOOP_THREE to 1e-11 relative
(1e-10 for BiCGStab, 1e-4 for the FP32 iterations of a mixed solve: rounding of
reordered sums, some 300 terms of a thread and a tree over 3e5 rows), and a
second solve without any memory gives the first one's x bit for bit."""
import numpy as np
import pytest

import synth
from helpers import share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_THREE

pytestmark = pytest.mark.gpu

MESHES = {
    # by rank 3 rows per thread and in one run 3: both cuts are tried
    "ranks": lambda: synth.small((70, 65, 62), ("blocks", 2, 1, 2), kappa=(1e-1, 1.0), seed=41),
    # no cut of its own numbering fits: an order is looked for
    "random": lambda: synth.small((68, 66, 64), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=42, scramble=True),
}
ALL = 2 ** 64 - 1


@pytest.mark.parametrize("mesh", sorted(MESHES))
def test_any_allocation_may_fail(mesh):
    torch = torch_mod()
    w = MESHES[mesh]()
    vals = share_values(w)
    b = dev_tensor(w.rhs())
    kinds = (dict(), dict(precision="mixed"), dict(method="bicgstab"))
    ref = []
    for kw in kinds:
        plan = make_plan(w)
        update(plan, vals)
        ref.append(plan.solve(b, tol=1e-13, max_iter=2, fused_loop=RP_LOOP_THREE, check=False, **kw)[0])
        plan.close()
    for faults in [1 << k for k in range(20)] + [ALL - (1 << k) + 1 for k in range(20)]:
        plan = make_plan(w)
        update(plan, vals)
        for kw, x3 in zip(kinds, ref):
            plan.set_loop_faults(faults)
            first = plan.solve(b, tol=1e-13, max_iter=2, check=False, **kw)[0]
            plan.set_loop_faults(ALL)
            again = plan.solve(b, tol=1e-13, max_iter=2, check=False, **kw)[0]
            plan.set_loop_faults(0)
            later = plan.solve(b, tol=1e-13, max_iter=2, check=False, **kw)[0]
            bar = 1e-11 if not kw else 1e-10 if "method" in kw else 1e-4
            for x in (first, again, later):
                assert float((x - x3).norm()) <= bar * float(x3.norm()), (mesh, hex(faults), kw)
            assert torch.equal(first, again), (mesh, hex(faults), kw)
        plan.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_small_systems_without_memory(precision):
    torch = torch_mod()
    w = synth.small((20, 19, 18), ("blocks", 2, 1, 1), kappa=(1e-1, 1.0), seed=43)
    plan = make_plan(w)
    update(plan, share_values(w))
    b = dev_tensor(w.rhs())
    ref = plan.solve(b, tol=1e-9, precision=precision, fused_loop=RP_LOOP_THREE)
    for faults in (1, 2, ALL, 0):
        plan.set_loop_faults(faults)
        got = plan.solve(b, tol=1e-9, precision=precision)
        assert torch.equal(got[0], ref[0]) and got[1] == ref[1], hex(faults)
    plan.close()
