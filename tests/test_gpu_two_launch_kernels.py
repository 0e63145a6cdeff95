"""The two-launch CG iteration where RP_LOOP_AUTO still takes it: small systems
whose rows are too long for the resident loop, and, without memory for that
loop's slots, any small system.  Bit for bit the three-launch iteration, over
the systems and budgets of test_gpu_two_launch.py."""
import pytest

import synth
from helpers import share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_AUTO, RP_LOOP_THREE
from test_gpu_two_launch import CASES, _same, _setup

pytestmark = pytest.mark.gpu

NO_MEMORY = 2 ** 64 - 1


def _both(plan, b, **kw):
    res = []
    x0 = kw.pop("x", None)
    for fl in (RP_LOOP_AUTO, RP_LOOP_THREE):
        plan.set_loop_faults(NO_MEMORY)
        res.append(plan.solve(b, x=None if x0 is None else x0.clone(), fused_loop=fl, check=False, **kw))
    _same(*res)
    return res[0]


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_rr"])
def test_without_the_resident_loop(name, precision):
    w = CASES[name]()
    _, _, plan = _setup(w)
    b = dev_tensor(w.rhs())
    x, info = _both(plan, b, tol=1e-8, precision=precision)
    assert info["status"] == 0
    for max_iter in (1, 2, 5, 37):
        for check_every in (1, 3, 32):
            _both(plan, b, tol=1e-13, precision=precision, max_iter=max_iter, check_every=check_every)
    plan.close()


@pytest.mark.parametrize("shape,stencil", [((64, 64, 64), 7), ((64, 64, 64), 27), ((45, 43, 41), 27), ((9, 3, 2), 27)])
@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_rr"])
def test_long_rows_and_the_largest(shape, stencil, precision):
    w = synth.small(shape, ("blocks", 2, 1, 1), kappa=(1e-1, 1.0), seed=95, stencil=stencil)
    plan = make_plan(w)
    update(plan, share_values(w))
    b = dev_tensor(w.rhs())
    if stencil == 27:   # no fault needed
        _same(plan.solve(b, tol=1e-8, precision=precision),
              plan.solve(b, tol=1e-8, precision=precision, fused_loop=RP_LOOP_THREE))
    _both(plan, b, tol=1e-8, precision=precision)
    _both(plan, b, x=torch_mod().ones_like(b), tol=1e-9, precision=precision)
    plan.close()
