"""The one-lane even-odd SAP phase (k_sap_phase_eo, k_bsap_phase_eo): FP16 and BF16 storage in the
even-odd site order at omega = 1.  Blocks at the edges of its rule: fewer sites than a wave, odd
numbers of sites, faces of more sites than the workgroup has threads (extent 2), the smallest
and largest of each LDS pitch, the largest block it takes and the first it leaves to the
two-lane kernel, and omega != 1, which it also leaves.  Tolerances are those of the M_SAP chain
in 16-bit storage (3 unit roundoffs: 1.5e-3 and 1.2e-2), the block inverse 2 (1e-3, 8e-3)."""
import numpy as np
import pytest

from paper_1210_7398_amd import synth
from tests.gpu_common import check_close, relerr, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = {"fp16": (1e-3, 1.5e-3), "bf16": (8e-3, 1.2e-2)}
EO = (0, 0, 0, 0)
# block: (lattice, omega)
BLOCKS = {(2, 2, 2, 2): ((4, 4, 4, 8), 1.0), (3, 3, 3, 3): ((6, 6, 6, 6), 1.0), (4, 4, 4, 4): ((8, 8, 8, 16), 1.0),
          (5, 4, 3, 6): ((10, 8, 6, 12), 1.0), (2, 4, 8, 8): ((4, 8, 16, 16), 1.0), (4, 8, 8, 4): ((8, 16, 16, 8), 1.0),
          (3, 7, 7, 7): ((6, 14, 14, 14), 1.0), (4, 4, 4, 6): ((8, 8, 8, 12), 1.2)}


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("B", list(BLOCKS), ids=lambda B: "x".join(map(str, B)))
def test_phase_parity(orc, B, prec):
    from paper_1210_7398_amd import sapq

    L, omega = BLOCKS[B]
    print(L, B, omega, prec, flush=True)
    kappa, bc = 0.125, (1, 1, 1, -1)
    U = synth.gauge_field(L, 0.25, 7)
    F = synth.clover_inverse(L, U, 1.0, kappa)
    s = sapq.Solver(L, B, EO, kappa, bc=bc, omega=omega, n_sap=3, prec=prec)
    s.load_gauge(to_dev(U))
    s.load_clover(to_dev(F))
    v = synth.gaussian_spinor(L, 301)
    prm = orc.params(kappa, n_sap=3, omega=omega)
    ts, tm = TOL[prec]
    for colour in (0, 1):
        want = orc.ssor(L, B, EO, U, F, prm, colour, v, bc=bc)
        check_close(to_host(s.ssor(to_dev(v), colour)), want, ts, f"SSOR colour {colour}")
    y_w, dy_w = orc.msap(L, B, EO, U, F, prm, v, bc=bc)
    y, dy = (to_host(t) for t in s.sap_precondition(to_dev(v)))
    check_close(y, y_w, tm, "M_SAP")
    check_close(dy, dy_w, tm, "D M_SAP")
    x, w = s.dk(to_dev(v))
    x_w, w_w = orc.dk(L, B, EO, U, F, prm, v, bc=bc)
    check_close(to_host(x), x_w, ts, "K")
    check_close(to_host(w), w_w, tm, "D K")


def test_batched_solve(orc):
    """Two fields of different size, blocks whose faces loop, to the oracle's true residual."""
    from paper_1210_7398_amd import sapq

    B, kappa, solvers, sources, fields = (2, 4, 4, 6), 0.125, [], [], []
    for L, n in (((4, 8, 8, 12), 3), ((8, 8, 16, 12), 1)):
        U = synth.gauge_field(L, 0.25, 7)
        F = synth.clover_inverse(L, U, 1.0, kappa)
        s = sapq.Solver(L, B, EO, kappa, prec="fp16", outer="defect")
        s.load_gauge(to_dev(U))
        s.load_clover(to_dev(F))
        solvers.append(s)
        fields.append((L, U, F))
        sources.append(np.stack([synth.gaussian_spinor(L, 40 + k) for k in range(n)]))
    xs, _ = sapq.solve_batch(solvers, [to_dev(b) for b in sources], tol=1e-10)
    for (L, U, F), b, x in zip(fields, sources, xs):
        for k in range(len(b)):
            assert relerr(orc.dslash(L, U, F, kappa, to_host(x[k])), b[k]) <= 1.001e-10
