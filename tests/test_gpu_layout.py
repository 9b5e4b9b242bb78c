"""Layout conversion of spinor fields (k_pack_spinor, k_unpack_spinor and their difference
form, and the operator's own output tile): with F = 0 the operator and M_SAP are the identity, so every call must return its input
exactly, rounded to the storage precision (to FP16 and BF16 directly or through FP32).  Sizes
around the kernels' tiles of 128 (FP64 operator: 64) sites: a lattice that ends inside a tile, blocks of fewer and of
more sites than a tile, odd extents."""
import numpy as np
import pytest
import torch

from paper_1210_7398_amd import sapq, synth

pytestmark = pytest.mark.gpu

SHAPES = [((6, 4, 4, 6), (3, 2, 2, 3), (0, 0, 0, 0)), ((6, 6, 6, 6), (3, 3, 3, 3), (0, 0, 0, 0)), ((8, 4, 4, 8), (4, 2, 2, 4), (2, 2, 2, 2)),
          ((10, 8, 6, 12), (5, 4, 3, 6), (0, 0, 0, 0)), ((12, 12, 12, 24), (6, 6, 6, 12), (3, 3, 3, 6))]


def check(got, v, prec):
    got, v = got.cpu().numpy().view(np.float64), v.view(np.float64)
    f = v.astype(np.float32)
    if prec == "fp64":
        ok = got == v
    elif prec == "fp32":
        ok = got == f
    elif prec == "fp16":
        ok = (got == v.astype(np.float16)) | (got == f.astype(np.float16))
    else:
        m, e = np.frexp(v)  # BF16 keeps 8 significant bits; rint rounds ties to even
        ok = (got == np.ldexp(np.rint(m * 256), e - 8)) | (got == torch.from_numpy(f).to(torch.bfloat16).double().numpy())
    assert ok.all(), (prec, int((~ok).sum()))


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("L, B, S", SHAPES)
def test_layout_round_trip(L, B, S, prec):
    print(L, B, S, prec, flush=True)
    V = int(np.prod(L))
    s = sapq.Solver(L, B, S, 0.125, prec=prec)
    s.load_gauge(torch.from_numpy(synth.unit_gauge(L)).cuda())
    s.load_clover(torch.zeros((V, 2, 6, 6), dtype=torch.complex128, device="cuda"))
    v = synth.gaussian_spinor(L, 5)
    vd = torch.from_numpy(v).cuda()
    for p in ("fp64", prec):
        check(s.dslash(vd, p), v, p)
    y, dy = s.sap_precondition(vd)
    check(y, v, prec)
    check(dy, v, prec)
