"""Solves in several threads, each on a plan and a stream of its own.  Small ones
share the device as launched kernels do: four threads finish in well under four
times a solve (0.9 of that while loops ran one after the other, 0.3 side by side).
Solves of all forms together, loops that fill the device among them, give what
each gives alone, bit for bit."""
import threading
import time

import pytest

import synth
from helpers import share_values
from gpu_util import dev_tensor, make_plan, update, torch_mod
from paper_2510_08536_amd import RP_LOOP_COOPERATIVE

pytestmark = pytest.mark.gpu


def _plan(shape, seed, bi=False):
    w = synth.small(shape, ("blocks", 2, 1, 2), kappa=(1e-1, 1.0), seed=seed)
    plan = make_plan(w)
    update(plan, share_values(w, values=w.momentum_values(pe=3.0)) if bi else share_values(w), lower=bi)
    return plan, dev_tensor(w.rhs())


def _together(jobs, reps):
    """reps solves of every job, a thread each; (seconds, what went wrong)"""
    torch = torch_mod()
    wrong, go = [], threading.Barrier(len(jobs) + 1)

    def work(plan, b, kw, ref):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                plan.solve(b, **kw)
                go.wait()
                for _ in range(reps):
                    if not torch.equal(plan.solve(b, **kw)[0], ref):
                        wrong.append(("differs", kw))
        except Exception as e:  # reported by the test's own thread
            wrong.append(repr(e))

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    go.wait()
    t0 = time.perf_counter()
    for t in threads:
        t.join()
    return time.perf_counter() - t0, wrong


def test_small_solves_share_the_device():
    torch = torch_mod()
    kw, reps = dict(tol=1e-8), 40
    jobs = []
    for k in range(4):
        plan, b = _plan((32, 32, 32), 71 + k)
        jobs.append((plan, b, kw, plan.solve(b, **kw)[0]))
    torch.cuda.synchronize()
    alone = together = 1e9
    for _ in range(3):   # the best of three: other work on the host only adds
        s, wrong = 0.0, []
        for j in jobs:
            t, w = _together([j], reps)
            s, wrong = s + t, wrong + w
        t, w = _together(jobs, reps)
        assert not wrong + w, wrong + w
        alone, together = min(alone, s), min(together, t)
    print(f"four solves one after the other {alone / reps * 1e3:.2f} ms, in four threads {together / reps * 1e3:.2f} ms")
    assert together <= 0.6 * alone
    for plan, *_ in jobs:
        plan.close()


def test_all_forms_together():
    torch = torch_mod()
    jobs = []
    for shape, seed, kw in (((20, 19, 18), 81, {}), ((64, 64, 64), 82, {}), ((64, 64, 64), 83, dict(precision="mixed")),
                            ((70, 66, 64), 84, {}), ((70, 66, 64), 85, dict(precision="mixed_rr")),
                            ((16, 16, 16), 86, dict(method="bicgstab")), ((70, 66, 64), 87, dict(method="bicgstab")),
                            ((30, 31, 32), 88, dict(fused_loop=RP_LOOP_COOPERATIVE)),
                            ((40, 40, 40), 89, dict(precond="amg"))):
        kw = dict(kw, tol=1e-8)
        plan, b = _plan(shape, seed, kw.get("method") == "bicgstab")
        jobs.append((plan, b, kw, plan.solve(b, **kw)[0]))
    torch.cuda.synchronize()
    _, wrong = _together(jobs, 6)
    assert not wrong, wrong
    for plan, *_ in jobs:
        plan.close()
