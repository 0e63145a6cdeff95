"""The one-launch loops where a wait for another workgroup's value ends first
(rp_plan_set_loop_faults bounds it at a few polls, so that workgroups leave at
any exchange, some of them after others have finished): the solve goes on with
launched kernels from the x at hand and meets its residual, the plan's next
solve takes launched kernels, bit for bit, and once the bound is lifted the
loop is back with the iterates it had."""
import numpy as np
import pytest

import oracle
import synth
from helpers import share_ranks, share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_THREE

pytestmark = pytest.mark.gpu

CG, BI = dict(kind="cg"), dict(kind="bi")
CASES = {
    "resident": ((33, 31, 30), ("blocks", 2, 1, 1), False, CG),
    "resident_large": ((64, 64, 64), ("blocks", 2, 2, 2), False, CG),
    "tile": ((70, 65, 62), ("blocks", 2, 1, 2), False, CG),
    "tile_order": ((68, 66, 64), ("blocks", 1, 1, 1), True, CG),
    "bi_two_tiles": ((27, 19, 1), ("blocks", 1, 1, 1), False, BI),
    "bi_short_halos": ((51, 52, 50), ("blocks", 2, 1, 2), False, BI),
    "bi_order": ((70, 66, 64), ("rcb", 3), True, BI),
    "bi_x_in_memory": ((98, 95, 96), ("blocks", 2, 2, 2), False, BI),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_goes_on_with_launches(name):
    import scipy.sparse as sp
    torch = torch_mod()
    shape, ranks, scramble, kind = CASES[name]
    w = synth.small(shape, ranks, kappa=(1e-1, 1.0), seed=51, scramble=scramble)
    bi = kind["kind"] == "bi"
    vals = share_values(w, values=w.momentum_values(pe=3.0)) if bi else share_values(w)
    m = oracle.merge(w.part.n_cells, 0, w.n_ranks, share_ranks(w))
    val64, *_ = oracle.update(m, oracle.receive_buffer(vals))
    A = sp.csr_matrix((val64, m.col, m.row_ptr), shape=(m.n_rows, m.n_rows))
    plan = make_plan(w)
    update(plan, vals, lower=bi)
    bh = w.rhs()
    b, x0 = dev_tensor(bh), np.random.default_rng(5).uniform(-1, 1, plan.n_rows)
    solves = ([dict(method="bicgstab"), dict(method="bicgstab", transpose=1)] if bi else
              [dict(), dict(precision="mixed"), dict(precision="mixed_rr")])
    for kw in solves:
        M = A.T if kw.get("transpose") else A
        for start in (None, x0):
            def solve(**more):
                return plan.solve(b, x=None if start is None else dev_tensor(start), tol=1e-8, **kw, **more)
            plan.set_loop_faults()
            loop, three = solve(), solve(fused_loop=RP_LOOP_THREE)
            for waits in (1, 2, 3, 8, 40, 200):
                print(name, kw, start is None, "waits", waits, flush=True)
                plan.set_loop_faults(0, waits)
                x, info = solve()
                rr = np.linalg.norm(bh - M @ x.cpu().numpy()) / np.linalg.norm(bh)
                assert info["status"] == 0 and rr <= 1e-8 * (1 + 1e-6), (name, kw, waits, info, rr)
                if waits == 1 and name != "bi_two_tiles":   # (two tiles may find each other's values at once)
                    after = solve()
                    assert torch.equal(after[0], three[0]) and after[1] == three[1], (name, kw)
            plan.set_loop_faults()
            again = solve()
            assert torch.equal(again[0], loop[0]) and again[1] == loop[1], (name, kw)
    plan.close()
