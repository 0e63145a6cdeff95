"""Updates that run without the host enqueueing them: an update captured in a
HIP graph runs again at every replay, with whatever values the caller's arrays
hold then.  A solve after a replay has to meet its residual on those values,
in every form that keeps something made from the values between solves: the
tiled loops' slices, A^T's values, the solve-order copy, the block-Jacobi
inverses and the multigrid's coarse matrices (the last two only precondition;
stale, they show in the iterates).  Checked against a second plan that
was given the same values by an update of its own: same kernels, same bits."""
import pytest

import synth
from helpers import share_values
from gpu_util import dev_tensor, make_plan, torch_mod

pytestmark = pytest.mark.gpu

SOLVES = {
    "cg_resident": ((20, 19, 18), {}),
    "cg_tile": ((70, 65, 62), {}),
    "cg_tile_mixed": ((70, 65, 62), dict(precision="mixed")),
    "bicgstab": ((70, 65, 62), dict(method="bicgstab")),
    "bicgstab_transposed": ((70, 65, 62), dict(method="bicgstab", transpose=1)),
    "solve_order": ((20, 19, 18), dict(order=1)),
    "solve_order_transposed": ((20, 19, 18), dict(order=1, method="bicgstab", transpose=1)),
    "block_jacobi": ((20, 19, 18), dict(precond="block_jacobi", block_size=4)),
    "amg": ((40, 39, 38), dict(precond="amg")),
}


@pytest.mark.parametrize("name", sorted(SOLVES))
def test_solves_follow_replays(name):
    torch = torch_mod()
    size, kw = SOLVES[name]
    kw = dict(kw)
    order = kw.pop("order", 0)
    w = synth.small(size, ("blocks", 2, 1, 2), kappa=(1e-2, 1.0), seed=31, timesteps=3)
    momentum = kw.get("method") == "bicgstab"

    def slots(t):
        v = share_values(w, values=w.momentum_values(t)) if momentum else share_values(w, t)
        return torch.cat([dev_tensor(a) for r in v for a in (r["diag"], r["upper"], r.get("lower", r["upper"]),
                                                             r["iface"])])

    plan, other = make_plan(w), make_plan(w)
    for p in (plan, other):
        p.set_solve_order(order)
    src = slots(0)
    plan.update_slots(src)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.update_slots(src)
    b = dev_tensor(w.rhs())
    for t, scale in ((0, 1.0), (1, 1.0), (2, 3.0), (2, 3.0), (0, 0.5)):
        src.copy_(slots(t) * scale)
        g.replay()
        torch.cuda.synchronize()
        other.update_slots(src.clone())
        (x, i), (y, j) = (p.solve(b, tol=1e-9, **kw) for p in (plan, other))
        assert i["status"] == j["status"] == 0
        assert torch.equal(x, y), (name, t, float((x - y).norm() / y.norm()))
        assert i["iters"] == j["iters"] and i["rel_res"] == j["rel_res"], (i, j)
    plan.close()
    other.close()
