"""Weight gradient of the learned stage on the FP32 matrix cores (k_nn_wgrad): lattices that end
inside a tile of 32 sites, fewer sites than one chunk per workgroup, chunks past the last site,
blocks of odd extents, both record types, against the FP64 oracle.  Only FP32 rounding of the
sums remains on the FP32 path (1e-4, as for the 8^4 gradient); the MFMA path rounds its
activations to BF16 (2e-2, likewise)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1210_7398_amd import sapq, synth

from gpu_common import check_close, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPES = [((4, 4, 4, 4), (2, 2, 2, 2)), ((6, 4, 4, 6), (3, 2, 2, 3)), ((10, 4, 6, 12), (5, 2, 3, 6)),
          ((12, 12, 12, 16), (6, 6, 6, 8))]


@pytest.mark.parametrize("nn_fp32, tol", [(True, 1e-4), (False, 2e-2)])
@pytest.mark.parametrize("L, B", SHAPES)
def test_weight_gradient_parity(L, B, nn_fp32, tol):
    print(L, B, nn_fp32, flush=True)
    bc = (1, 1, 1, -1)
    U = synth.gauge_field(L, 0.25, 7)
    rng = np.random.default_rng(3)
    w = torch.from_numpy(0.1 * rng.normal(size=sapq.nn_param_count())).to(torch.bfloat16).float()
    s = sapq.Solver(L, B, (0, 0, 0, 0), 0.125, bc=bc, nn=True, nn_fp32=nn_fp32)
    s.load_gauge(to_dev(U))
    s.nn_set_weights(w.cuda())
    r, gz = synth.gaussian_spinor(L, 21), synth.gaussian_spinor(L, 22)
    gw, gin = s.nn_backward(to_dev(gz), to_dev(r))
    Ws = oracle.nn_unflatten(w.double().numpy())
    grads, gin_w = oracle.nn_backward(L, U, Ws, r, gz, bc)
    want, got = oracle.nn_flatten(grads), gw.cpu().double().numpy()
    off = 0
    for ci, co in ((1, 8), (8, 8), (8, 1)):  # each layer by itself
        n = 2 * 16 * 9 * ci * co
        e = np.linalg.norm(got[off:off + n] - want[off:off + n]) / np.linalg.norm(want[off:off + n])
        print(f"layer {ci}->{co}: {e:.2e} (tol {tol:.0e})")
        assert e < tol
        off += n
    check_close(to_host(gin), gin_w, 1e-5 if nn_fp32 else 2e-2, "input gradient")
