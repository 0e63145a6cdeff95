"""Products at the edges of their launch rules: rows longer than a group's LDS
(more than eight entries on average) just below, at and past the 2048 row groups
that run at once, from where blocks loop; y just below and past the size stored
non-temporally, in both precisions.  Band matrices, bit for bit against the same
sums in numpy (row sums from 0 in column order, one rounding per product and sum).
CG of long rows past the size of the folded sums, which they do not take:
iterates after three iterations to 1e-11 relative (sums of 4 million terms in
another order)."""
import numpy as np
import pytest

from gpu_util import assert_bits_equal, dev_tensor
from paper_2510_08536_amd import Plan, RP_LOOP_THREE

pytestmark = pytest.mark.gpu


class Band:
    """diagonal, and k off-diagonals on either side"""

    def __init__(self, n, k, seed):
        g = np.random.default_rng(seed)
        self.n, self.k = n, k
        self.off = [-g.uniform(0.1, 1.0, n - j) for j in range(1, k + 1)]
        self.diag = np.full(n, 0.1)
        for j, o in enumerate(self.off, 1):
            self.diag[:-j] -= o
            self.diag[j:] -= o
        own = np.repeat(np.arange(n, dtype=np.int32), k).reshape(n, k)
        nbr = own + np.arange(1, k + 1, dtype=np.int32)
        ok = nbr < n
        up = np.zeros((n, k))
        for j, o in enumerate(self.off, 1):
            up[:n - j, j - 1] = o
        z = np.zeros(0, np.int32)
        self.plan = Plan([n], 0, 1, [dict(owner=own[ok], neighbour=nbr[ok], iface_cell=z, iface_nbr_rank=z,
                                          iface_nbr_cell=z)])
        self.plan.update([self.diag], [up[ok]], [np.zeros(0)])

    def mul(self, x):
        y = np.zeros_like(x)
        for j in range(self.k, 0, -1):
            y[j:] = y[j:] + self.off[j - 1].astype(x.dtype) * x[:-j]
        y = y + self.diag.astype(x.dtype) * x
        for j in range(1, self.k + 1):
            y[:-j] = y[:-j] + self.off[j - 1].astype(x.dtype) * x[j:]
        return y


@pytest.mark.parametrize("n,k", [(2048 * 256, 4), (2048 * 256 + 1, 4), (2048 * 256 + 70001, 6), (2048 * 256 + 1, 3),
                                 (1 << 21, 1), ((1 << 21) + 1, 1), (1 << 22, 1), ((1 << 22) + 1, 1)])
def test_products_to_the_bit(n, k):
    m = Band(n, k, n)
    x = np.random.default_rng(1).uniform(-1, 1, n)
    for dtype in (np.float64, np.float32):
        xv = x.astype(dtype)
        assert_bits_equal(m.plan.spmv(dev_tensor(xv)).cpu().numpy(), m.mul(xv), f"n {n}, band {k}, {dtype.__name__}")
    m.plan.close()


def test_long_rows_without_the_fold():
    m = Band((1 << 22) + 300, 4, 5)
    b = np.random.default_rng(2).uniform(-1, 1, m.n)
    x, r = np.zeros(m.n), b.copy()
    p = r / m.diag
    rz = r @ p
    for _ in range(3):
        q = m.mul(p)
        a = rz / (p @ q)
        x += a * p
        r -= a * q
        s = r / m.diag
        rz, old = r @ s, rz
        p = s + (rz / old) * p
    xg, info = m.plan.solve(dev_tensor(b), tol=1e-14, max_iter=3, fused_loop=RP_LOOP_THREE, check=False)
    assert info["iters"] == 3
    assert np.linalg.norm(xg.cpu().numpy() - x) <= 1e-11 * np.linalg.norm(x)
    m.plan.close()
