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


VARIANTS = {"mixed": dict(precision="mixed"), "mixed_rr": dict(precision="mixed_rr"), "graph": dict(graph=1),
            "block_jacobi_lanes": dict(precond="block_jacobi", block_size=4),
            "block_jacobi": dict(precond="block_jacobi", block_size=3), "amg": dict(precond="amg"),
            "amg_mixed": dict(precond="amg", precision="mixed")}


def _chain(n):
    """off-diagonals -1, diagonal 2.1 but for the ends: the same system at any length"""
    z = np.zeros(0, np.int32)
    own = np.arange(n - 1, dtype=np.int32)
    plan = Plan([n], 0, 1, [dict(owner=own, neighbour=own + 1, iface_cell=z, iface_nbr_rank=z, iface_nbr_cell=z)])
    plan.update([np.full(n, 2.1)], [np.full(n - 1, -1.0)], [np.zeros(0)])
    return plan, dev_tensor(np.random.default_rng(7).uniform(-1, 1, n))


@pytest.mark.parametrize("name", sorted(VARIANTS))
def test_other_readers_of_the_sums(name):
    """Every other kernel that reads the folded sums: a solve of the first size
    with the fold meets its residual in the iterations that the last size without
    takes (four rows more of 4 million: the same convergence, two for rounding)."""
    iters = []
    for n in (GROUPS * 256, GROUPS * 256 + 4):
        plan, b = _chain(n)
        x, info = plan.solve(b, tol=1e-9, fused_loop=RP_LOOP_THREE, **VARIANTS[name])
        assert info["status"] == 0 and float((b - plan.spmv(x)).norm()) <= 1e-9 * (1 + 1e-6) * float(b.norm())
        iters.append(info["iters"])
        plan.close()
    assert abs(iters[0] - iters[1]) <= 2, iters
