"""Three-launch CG on the largest systems, where the product's blocks take one
row group each and their sums are folded by a launch of their own: the last
size without and the first with it, and a ragged one, against CG in numpy on
the same chain.  Iterates after a fixed budget agree to 1e-11 relative (sums of
4 million terms in another order, some 1e-13, through three iterations)."""
import numpy as np
import pytest

from gpu_util import dev_tensor
from paper_2510_08536_amd import Plan, RP_LOOP_THREE

pytestmark = pytest.mark.gpu

GROUPS = 16384   # row groups of 256 up to which the blocks loop


@pytest.mark.parametrize("n", [GROUPS * 256, GROUPS * 256 + 1, GROUPS * 256 + 70001])
def test_iterates_match_numpy(n):
    g = np.random.default_rng(n)
    off = -g.uniform(0.1, 1.0, n - 1)
    diag = np.full(n, 0.1)
    diag[:-1] -= off
    diag[1:] -= off
    z = np.zeros(0, np.int32)
    own = np.arange(n - 1, dtype=np.int32)
    plan = Plan([n], 0, 1, [dict(owner=own, neighbour=own + 1, iface_cell=z, iface_nbr_rank=z, iface_nbr_cell=z)])
    plan.update([diag], [off], [np.zeros(0)])
    b = g.uniform(-1, 1, n)

    def mul(v):
        y = diag * v
        y[:-1] += off * v[1:]
        y[1:] += off * v[:-1]
        return y

    x, r = np.zeros(n), b.copy()
    p = r / diag
    rz = r @ p
    for _ in range(3):
        q = mul(p)
        a = rz / (p @ q)
        x += a * p
        r -= a * q
        s = r / diag
        rz, old = r @ s, rz
        p = s + (rz / old) * p
    xg, info = plan.solve(dev_tensor(b), tol=1e-14, max_iter=3, fused_loop=RP_LOOP_THREE, check=False)
    assert info["iters"] == 3
    assert np.linalg.norm(xg.cpu().numpy() - x) <= 1e-11 * np.linalg.norm(x)
    plan.close()
