"""The LDS limit of the batched phase kernels, which every batch of a process shares: a program
that asks for the work memory of a batch with smaller blocks (or solves one) in another thread
may not take away the LDS that a running batch launches with."""
import ctypes
import threading

import pytest

from paper_1210_7398_amd import synth
from tests.gpu_common import relerr, to_dev, to_host

pytestmark = pytest.mark.gpu

# order, blocks of the solved batch and of the other, their precision: the one-lane kernel (both
# blocks in the pitch of 1026) and the two-lane kernel
CASES = [((0, 0, 0, 0), (4, 4, 8, 8), (4, 4, 6, 6), "fp16"), ((2, 2, 2, 2), (4, 4, 8, 8), (4, 4, 6, 8), "fp32")]


def _solver(L, B, S, kappa, prec):
    from paper_1210_7398_amd import sapq

    U = synth.gauge_field(L, 0.25, 7)
    F = synth.clover_inverse(L, U, 1.0, kappa)
    s = sapq.Solver(L, B, S, kappa, prec=prec, outer="defect")
    s.load_gauge(to_dev(U))
    s.load_clover(to_dev(F))
    return s, U, F


@pytest.mark.parametrize("S, B, B2, prec", CASES, ids=["one-lane", "two-lane"])
def test_smaller_batch_in_another_thread(orc, S, B, B2, prec):
    from paper_1210_7398_amd import sapq

    kappa, L = 0.12, tuple(2 * b for b in B)
    print(B, B2, prec, flush=True)
    s, U, F = _solver(L, B, S, kappa, prec)
    other, _, _ = _solver(tuple(2 * b for b in B2), B2, S, kappa, prec)
    src = synth.gaussian_spinor(L, 70)[None]
    ctxs, nrhs = (ctypes.c_void_p * 1)(other.h), (ctypes.c_int * 1)(1)
    stop, calls = threading.Event(), [0]

    def ask():
        while not stop.is_set():
            assert sapq.lib().sapq_batch_arena_bytes(ctxs, 1, nrhs) > 0
            calls[0] += 1

    t = threading.Thread(target=ask)
    t.start()
    try:
        # another tolerance each time: the batch's graphs are captured anew
        for k in range(30):
            tol = 1e-10 * (1 - 0.01 * k)
            (x,), _ = sapq.solve_batch([s], [to_dev(src)], tol=tol)
            assert relerr(orc.dslash(L, U, F, kappa, to_host(x[0])), src[0]) <= 1.001 * tol
    finally:
        stop.set()
        t.join()
    assert calls[0] > 30
