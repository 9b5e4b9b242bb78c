"""What is not finite stays so in the one-lane even-odd phase, which takes the even sites' residual for
zero: a source with one value that is not a number, infinite or too large for FP16 gives results
that are not finite at the same components as in the two-lane kernel, which computes that residual (a
relaxation that FP64 tells from 1 and FP32 does not takes it)."""
import math

import pytest

from paper_1210_7398_amd import synth
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu

EO = (0, 0, 0, 0)


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("n_ssor, n_sap", [(1, 1), (2, 3)])
@pytest.mark.parametrize("B", [(4, 4, 4, 4), (5, 4, 3, 6), (4, 4, 8, 8)], ids=lambda B: "x".join(map(str, B)))
def test_not_finite(B, n_ssor, n_sap, prec):
    import torch

    from paper_1210_7398_amd import sapq

    L = (4 * B[0],) + tuple(2 * b for b in B[1:])
    print(L, B, n_ssor, n_sap, prec, flush=True)
    U = synth.gauge_field(L, 0.25, 7)
    F = synth.clover_inverse(L, U, 1.0, 0.125)
    v = to_dev(synth.gaussian_spinor(L, 307))
    solvers = []
    for omega in (1.0, 1.0 + 1e-12):
        s = sapq.Solver(L, B, EO, 0.125, omega=omega, n_ssor=n_ssor, n_sap=n_sap, prec=prec)
        s.load_gauge(to_dev(U))
        s.load_clover(to_dev(F))
        solvers.append(s)
    for value in (math.nan, math.inf, 1e5):
        for site in (0, 1, math.prod(L) // 3):
            w = v.clone()
            w[site, 1, 1] = value
            got, want = ([torch.isfinite(torch.view_as_real(t)) for t in (*s.sap_precondition(w), *s.dk(w))] for s in solvers)
            for a, b in zip(got, want):
                assert torch.equal(a, b), (value, site, int((a & ~b).sum()))
