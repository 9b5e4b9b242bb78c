"""Small blocks in the even-odd order and 16-bit storage.  Up to 96 sites they take the two-lane
kernel, as at a relaxation that FP64 tells from 1 and FP32 does not, where the one-lane kernel is
out of the question and the arithmetic is that of omega = 1: the same bits.  From there on the
one-lane kernel: its smallest block, an odd number of sites, faces of more sites than it has
threads; against the oracle (tolerances of the M_SAP chain: 3 unit roundoffs, 1.5e-3 and 1.2e-2)."""
import pytest

from paper_1210_7398_amd import synth
from tests.gpu_common import check_close, to_dev, to_host

pytestmark = pytest.mark.gpu

EO = (0, 0, 0, 0)


def _solver(L, B, U, F, prec, **kw):
    from paper_1210_7398_amd import sapq

    s = sapq.Solver(L, B, EO, 0.125, prec=prec, **kw)
    s.load_gauge(to_dev(U))
    s.load_clover(to_dev(F))
    return s


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("B", [(2, 2, 2, 2), (2, 2, 2, 4), (3, 3, 3, 3), (2, 3, 4, 4)], ids=lambda B: "x".join(map(str, B)))
def test_up_to_96_sites_two_lane(B, prec):
    import torch

    L = tuple(4 * b for b in B)
    print(L, B, prec, flush=True)
    U = synth.gauge_field(L, 0.25, 7)
    F = synth.clover_inverse(L, U, 1.0, 0.125)
    v = to_dev(synth.gaussian_spinor(L, 305))
    a, b = (_solver(L, B, U, F, prec, omega=w).sap_precondition(v) for w in (1.0, 1.0 + 1e-12))
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("prec, tol", [("fp16", 1.5e-3), ("bf16", 1.2e-2)])
@pytest.mark.parametrize("B", [(3, 3, 3, 4), (2, 4, 4, 4), (3, 3, 3, 5)], ids=lambda B: "x".join(map(str, B)))
def test_above_96_sites(orc, B, prec, tol):
    L = tuple(2 * b for b in B)
    print(L, B, prec, flush=True)
    U = synth.gauge_field(L, 0.25, 7)
    F = synth.clover_inverse(L, U, 1.0, 0.125)
    v = synth.gaussian_spinor(L, 306)
    s = _solver(L, B, U, F, prec, n_sap=3)
    y_w, dy_w = orc.msap(L, B, EO, U, F, orc.params(0.125, n_sap=3), v)
    y, dy = (to_host(t) for t in s.sap_precondition(to_dev(v)))
    check_close(y, y_w, tol, "M_SAP")
    check_close(dy, dy_w, tol, "D M_SAP")
