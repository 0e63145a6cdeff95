"""The resident CG loop (RP_LOOP_AUTO on small systems with at most 8 entries
per row) against the three-launch iteration, bit for bit, at the sizes where
its shape changes: one row, the ends of a wavefront, of a row group and of a
workgroup, the first size past the smaller FP64 workgroup, and the largest;
budgets of one iteration and more, warm starts, and several plans at once on
streams of their own."""
import threading

import numpy as np
import pytest

import synth
from helpers import share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_AUTO, RP_LOOP_THREE, RP_LOOP_TWO_MAX_ROWS

pytestmark = pytest.mark.gpu

# rows: mesh
SIZES = {1: (1, 1, 1), 2: (2, 1, 1), 63: (63, 1, 1), 64: (8, 8, 1), 65: (13, 5, 1), 255: (17, 5, 3), 256: (8, 8, 4),
         257: (257, 1, 1), 511: (73, 7, 1), 513: (27, 19, 1), 1023: (33, 31, 1), 1025: (41, 5, 5),
         131072: (64, 64, 32), 131073: (43691, 3, 1), 262143: (87381, 3, 1), 262144: (64, 64, 64)}


@pytest.mark.parametrize("rows", sorted(SIZES))
def test_equals_three_launches(rows):
    torch = torch_mod()
    w = synth.small(SIZES[rows], ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=rows)
    plan = make_plan(w)
    assert plan.n_rows == rows <= RP_LOOP_TWO_MAX_ROWS
    update(plan, share_values(w))
    b = dev_tensor(w.rhs())
    x0 = dev_tensor(np.random.default_rng(rows).uniform(-1, 1, rows))
    for precision in ("fp64", "mixed", "mixed_rr"):
        for budget in (1, 23):
            for start in (None, x0):
                res = [plan.solve(b, x=None if start is None else start.clone(), tol=1e-13, max_iter=budget,
                                  precision=precision, fused_loop=fl, check=False)
                       for fl in (RP_LOOP_AUTO, RP_LOOP_THREE)]
                assert torch.equal(res[0][0], res[1][0]), (rows, precision, budget, start is None)
                assert res[0][1] == res[1][1], (res[0][1], res[1][1])
    plan.close()


def test_plans_on_streams_of_their_own():
    torch = torch_mod()
    plans = []
    for k in range(3):
        w = synth.small((40 + k, 36, 38), ("blocks", 2, 1, 2), kappa=(1e-1, 1.0), seed=40 + k)
        plan = make_plan(w)
        update(plan, share_values(w))
        b = dev_tensor(w.rhs())
        plans.append((plan, b, plan.solve(b, tol=1e-8)[0]))
    torch.cuda.synchronize()
    wrong = []

    def work(plan, b, ref):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(5):
                    if not torch.equal(plan.solve(b, tol=1e-8)[0], ref):
                        wrong.append("differs")
        except Exception as e:  # reported below, in the test's own thread
            wrong.append(repr(e))

    threads = [threading.Thread(target=work, args=p) for p in plans]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
    for plan, *_ in plans:
        plan.close()
