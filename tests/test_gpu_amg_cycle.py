"""The V-cycle's composed lists and its one-workgroup tail at their edges, bit
for bit against the oracle's V-cycle: a tail that starts on an odd or an even
level, right at level 1, with vectors in LDS and (hierarchies that coarsen by
17 rows a level: a chain of growing couplings, 16 matching rounds) in memory."""
import numpy as np
import pytest

import oracle
import synth
from helpers import share_values, oracle_system
from gpu_util import dev_tensor, make_plan, update, assert_bits_equal

pytestmark = pytest.mark.gpu


def _chain(n, growth):
    w = synth.small((n, 1, 1), ("blocks", 5, 1, 1), kappa=(0.5, 1.0), seed=29, walls=(True, False, False))
    w.kappa0 = growth ** np.arange(w.kappa0.shape[0])
    return w


# name: system, first level of at most 1024 rows (the tail's)
CASES = {
    "chain_500": (lambda: _chain(500, 1.05), 1),
    "chain_230": (lambda: _chain(230, 1.1), 1),
    "tail_2": (lambda: synth.small((17, 16, 16), ("blocks", 2, 2, 1), kappa=(1e-2, 1.0), seed=31), 2),
    "tail_4": (lambda: synth.small((23, 20, 25), ("blocks", 2, 1, 3), kappa=(1e-2, 1.0), seed=32), 4),
    "tail_odd": (lambda: synth.small((19, 18, 23), ("rcb", 5), kappa=(1e-1, 1.0), seed=33, scramble=True), 3),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_vcycle_bit_exact(name):
    make, first = CASES[name]
    w = make()
    m, _, v64, *_ = oracle_system(w)
    h = oracle.AmgHierarchy(m, v64)
    sizes = [h.level_size(l) for l in range(h.n_levels)]
    assert next(l for l in range(1, len(sizes)) if sizes[l] <= 1024) == first, sizes
    plan = make_plan(w)
    update(plan, share_values(w))
    plan.amg_setup()
    rng = np.random.default_rng(8)
    for _ in range(2):
        r = rng.uniform(-1, 1, m.n_rows)
        assert_bits_equal(plan.amg_apply(dev_tensor(r)).cpu().numpy(), h.vcycle(r), name)
    b = w.rhs()
    for precision in ("fp64",) if name.startswith("chain") else ("fp64", "mixed"):
        x, info = plan.solve(dev_tensor(b), tol=1e-8, precision=precision, precond="amg")
        assert info["status"] == 0 and oracle.true_relres(m, v64, b, x.cpu().numpy()) <= 1e-8, (name, precision, info)
    plan.close()
