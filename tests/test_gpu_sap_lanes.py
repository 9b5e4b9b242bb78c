"""The SAP phase kernel's lane forms (k_sap_phase_parts): hyperplanes by four lanes per site and by
two, in one and in several passes, whole blocks alone on their CUs and sharing them, and a split
block whose halo wave also updates sites and copies more than 64 words.  Tolerances: FP32 2e-5
(its roundings through n_sap 3), 16-bit storage those of the M_SAP chain (block inverse 2, chain 3
unit roundoffs)."""
import numpy as np
import pytest

from paper_1210_7398_amd import synth
from tests.gpu_common import check_close, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = {"fp32": (2e-5, 2e-5), "fp16": (1e-3, 1.5e-3), "bf16": (8e-3, 1.2e-2)}
# lattice, block, sub-block, omega: planes of 1 to 6 sites; planes of 16 to 96 sites; of up to
# 304 (192 go by four lanes, 384 in one pass of two); of 264 in an odd shape; of 648 (several
# passes); omega with the (1 - omega) x term; more blocks than CUs; a split block
CASES = [((4, 4, 4, 4), (2, 2, 2, 2), (2, 2, 2, 2), 1.0), ((8, 8, 8, 8), (4, 4, 4, 4), (2, 2, 2, 2), 1.0),
         ((12, 12, 12, 12), (6, 6, 6, 6), (3, 3, 3, 3), 1.0), ((12, 8, 20, 12), (6, 4, 10, 6), (3, 2, 5, 3), 1.0),
         ((12, 12, 12, 12), (6, 6, 6, 6), (0, 0, 0, 0), 1.0), ((8, 12, 16, 8), (4, 6, 8, 4), (2, 3, 4, 2), 1.2),
         ((8, 8, 16, 16), (2, 2, 2, 2), (2, 2, 2, 2), 1.0), ((16, 16, 12, 12), (8, 8, 6, 6), (2, 2, 3, 3), 1.0)]


# (16-bit storage takes another kernel in the even-odd order)
PARAMS = [(*c, p) for c in CASES for p in TOL if any(c[2]) or p == "fp32"]


@pytest.mark.parametrize("L, B, S, omega, prec", PARAMS)
def test_phase_parity(orc, L, B, S, omega, prec):
    from paper_1210_7398_amd import sapq

    print(L, B, S, omega, prec, flush=True)
    kappa, bc = 0.125, (1, 1, 1, -1)
    U = synth.gauge_field(L, 0.25, 11)
    F = synth.clover_inverse(L, U, 1.0, kappa)
    s = sapq.Solver(L, B, S, kappa, bc=bc, omega=omega, n_sap=3, prec=prec)
    s.load_gauge(to_dev(U))
    s.load_clover(to_dev(F))
    v = synth.gaussian_spinor(L, 302)
    prm = orc.params(kappa, n_sap=3, omega=omega)
    ts, tm = TOL[prec]
    for colour in (0, 1):
        want = orc.ssor(L, B, S, U, F, prm, colour, v, bc=bc)
        check_close(to_host(s.ssor(to_dev(v), colour)), want, ts, f"SSOR colour {colour}")
    y_w, dy_w = orc.msap(L, B, S, U, F, prm, v, bc=bc)
    y, dy = (to_host(t) for t in s.sap_precondition(to_dev(v)))
    check_close(y, y_w, tm, "M_SAP")
    check_close(dy, dy_w, tm, "D M_SAP")


# the even-odd MR kernel's passes over a parity: the largest block of one pass (384 sites of a
# parity), the smallest sizes past it, the largest of two passes (768) and one of three
@pytest.mark.parametrize("B", [(4, 6, 4, 8), (4, 4, 7, 7), (4, 6, 8, 8), (5, 6, 7, 8)], ids=lambda B: "x".join(map(str, B)))
def test_eomr_passes(orc, B):
    from paper_1210_7398_amd import sapq

    L, kappa = tuple(2 * b for b in B), 0.125
    print(L, B, flush=True)
    U = synth.gauge_field(L, 0.25, 11)
    F = synth.clover_inverse(L, U, 1.0, kappa)
    s = sapq.Solver(L, B, (0, 0, 0, 0), kappa, n_sap=2, block_solver="eomr")
    s.load_gauge(to_dev(U))
    s.load_clover(to_dev(F))
    v = synth.gaussian_spinor(L, 303)
    y_w, dy_w = orc.msap(L, B, (0, 0, 0, 0), U, F, orc.params(kappa, n_sap=2, block_solver=1), v)
    y, dy = (to_host(t) for t in s.sap_precondition(to_dev(v)))
    check_close(y, y_w, 2e-5, "EO-MR M_SAP")
    check_close(dy, dy_w, 2e-5, "EO-MR D M_SAP")
