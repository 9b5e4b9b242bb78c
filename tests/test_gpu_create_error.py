"""An error that some earlier HIP call of the program left behind is not the context's: sapq_create
reports its own calls' results (blocks whose kernels need no raised LDS limit)."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
def test_create_after_a_foreign_error(prec):
    import torch

    from paper_1210_7398_amd import sapq

    lib = sapq.lib()
    s = sapq.Solver((8, 8, 8, 8), (4, 4, 4, 4), (0, 0, 0, 0), 0.12, prec=prec)
    arena = torch.empty_like(s.arena)
    torch.cuda.synchronize()
    h = ctypes.c_void_p()
    assert lib.hipSetDevice(-1) != 0  # refused on the host: no such device
    try:
        rc = lib.sapq_create(ctypes.byref(s.geom), ctypes.byref(s.params), ctypes.c_void_p(arena.data_ptr()),
                             arena.numel(), ctypes.c_void_p(s.stream.cuda_stream), ctypes.byref(h))
    finally:
        lib.hipGetLastError()
    assert rc == 0, lib.sapq_last_error()
    lib.sapq_destroy(h)
