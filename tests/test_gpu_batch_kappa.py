"""The batched solver at hopping parameters that FP32 does not hold (0.12, 0.1234), a different one
per field: its FP64 residual has to be that of the operator in FP64, so the oracle's true
residual is the one asked for (1e-10, with 0.1% for its own rounding; kappa rounded to FP32
is off by 1e-8 and more).  The three orders and splits that the batched phase kernels take."""
import numpy as np
import pytest

from paper_1210_7398_amd import synth
from tests.gpu_common import relerr, to_dev, to_host

pytestmark = pytest.mark.gpu

FIELDS = [((8, 8, 8, 8), 0.12, 2), ((8, 8, 8, 16), 0.1234, 1)]


@pytest.mark.parametrize("S, prec", [((2, 2, 2, 2), "fp32"), ((0, 0, 0, 0), "fp32"), ((0, 0, 0, 0), "fp16")])
def test_true_residual(orc, S, prec):
    from paper_1210_7398_amd import sapq

    print(S, prec, flush=True)
    solvers, sources, fields = [], [], []
    for L, kappa, n in FIELDS:
        U = synth.gauge_field(L, 0.25, 7)
        F = synth.clover_inverse(L, U, 1.0, kappa)
        s = sapq.Solver(L, (4, 4, 4, 4), S, kappa, prec=prec, outer="defect")
        s.load_gauge(to_dev(U))
        s.load_clover(to_dev(F))
        solvers.append(s)
        fields.append((L, kappa, U, F))
        sources.append(np.stack([synth.gaussian_spinor(L, 60 + k) for k in range(n)]))
    xs, stats = sapq.solve_batch(solvers, [to_dev(b) for b in sources], tol=1e-10)
    for (L, kappa, U, F), b, x in zip(fields, sources, xs):
        for k in range(len(b)):
            assert relerr(orc.dslash(L, U, F, kappa, to_host(x[k])), b[k]) <= 1.001e-10, (L, kappa, k)
