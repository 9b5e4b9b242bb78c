"""Blocks at the limit of a workgroup's LDS (160 KB): the largest iterates that the two-lane phase
kernel holds, whole and split, which a context has to accept although the even-odd MR kernel's
sums no longer fit beside them, and the largest block of that kernel with the first it refuses.
Tolerances: FP32 2e-5 (its roundings through n_sap 2), FP16 those of the M_SAP chain (3 unit roundoffs)."""
import pytest

from paper_1210_7398_amd import synth
from tests.gpu_common import check_close, to_dev, to_host

pytestmark = pytest.mark.gpu

EO = (0, 0, 0, 0)
# 1705 and 1701 sites in one workgroup (163,776 and 163,392 bytes), 1134 + 567 halo sites in each
# of two
CASES = [((1, 5, 11, 31), EO, "two-lane"), ((9, 9, 7, 3), (9, 9, 7, 3), "two-lane"), ((9, 9, 7, 4), (3, 3, 7, 2), "two-lane split")]


def _fields(L):
    U = synth.gauge_field(L, 0.25, 11)
    return U, synth.clover_inverse(L, U, 1.0, 0.125)


def _msap(orc, B, S, prec, tol, block_solver="ssor"):
    from paper_1210_7398_amd import sapq

    L = tuple(2 * b for b in B)
    print(L, B, S, prec, block_solver, flush=True)
    U, F = _fields(L)
    s = sapq.Solver(L, B, S, 0.125, n_sap=2, prec=prec, block_solver=block_solver)
    s.load_gauge(to_dev(U))
    s.load_clover(to_dev(F))
    v = synth.gaussian_spinor(L, 304)
    y_w, dy_w = orc.msap(L, B, S, U, F, orc.params(0.125, n_sap=2, block_solver=int(block_solver == "eomr")), v)
    y, dy = (to_host(t) for t in s.sap_precondition(to_dev(v)))
    check_close(y, y_w, tol, "M_SAP")
    check_close(dy, dy_w, tol, "D M_SAP")
    return s


@pytest.mark.parametrize("prec, tol", [("fp32", 2e-5), ("fp16", 1.5e-3)])
@pytest.mark.parametrize("B, S, kernel", CASES, ids=lambda p: "x".join(map(str, p)) if isinstance(p, tuple) else None)
def test_largest_blocks(orc, B, S, kernel, prec, tol):
    assert _msap(orc, B, S, prec, tol).phase_kernel == kernel


def test_largest_block_of_the_mr_solver(orc):
    from paper_1210_7398_amd import sapq

    _msap(orc, (2, 3, 1, 283), EO, "fp32", 2e-5, "eomr")  # 1698 sites
    with pytest.raises(sapq.SapqError, match="block too large"):
        sapq.Solver((10, 8, 10, 34), (5, 4, 5, 17), EO, 0.125, block_solver="eomr")  # 1700
