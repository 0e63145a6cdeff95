"""The slot gradient's work items (a face's two slots are one) at the edges of
its chunks, bit for bit against the oracle: ranks and regions that end inside,
at and past a block's 1024 items, ranks of one cell (no faces, only
interfaces), many small ranks in one chunk, and a share whose ranks have no
interface."""
import numpy as np
import pytest

import oracle
import synth
from helpers import share_ranks
from gpu_util import dev_tensor, make_plan, update, assert_bits_equal
from helpers import share_values

pytestmark = pytest.mark.gpu

CASES = {
    "one_cell": lambda: synth.small((1, 1, 1), ("blocks", 1, 1, 1), seed=1),
    "one_cell_ranks": lambda: synth.small((7, 3, 2), ("blocks", 7, 3, 2), kappa=(1e-1, 1.0), seed=2),
    "many_small_ranks": lambda: synth.small((24, 20, 3), ("rcb", 180), kappa=(1e-1, 1.0), seed=3),
    "no_interface": lambda: synth.small((16, 16, 16), ("blocks", 1, 1, 1), kappa=(1e-1, 1.0), seed=4),
    "cells_fill_a_chunk": lambda: synth.small((32, 32, 4), ("blocks", 1, 1, 4), kappa=(1e-1, 1.0), seed=5),
    "ragged": lambda: synth.small((19, 17, 23), ("rcb", 5), kappa=(1e-1, 1.0), seed=6, scramble=True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_bit_exact(name):
    w = CASES[name]()
    m = oracle.merge(w.part.n_cells, 0, w.n_ranks, share_ranks(w))
    plan = make_plan(w)
    update(plan, share_values(w))
    rng = np.random.default_rng(3)
    lam, x = rng.uniform(-1, 1, m.n_rows), rng.uniform(-1, 1, m.n_rows)
    g = plan.value_grad(dev_tensor(lam), dev_tensor(x)).cpu().numpy()
    assert_bits_equal(g, oracle.value_grad(m, lam, x), name)
    plan.close()
