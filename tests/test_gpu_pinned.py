"""Field copies to and from pinned host memory."""
import ctypes as C

import numpy as np
import pytest

from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu


# unpadded rows (37), padded ones in less than one piece of the pageable copies (60)
# and in several (250); the guard after the array stays as it was
@pytest.mark.parametrize("n", [(37, 11, 6), (60, 7, 5), (250, 41, 130)])
def test_pinned_round_trip(n):
    import torch
    from paper_0802_3775_amd import fdtd
    ncell = n[0] * n[1] * n[2]
    plan = fdtd.Plan(W.homogeneous_box(n, steps=1), max_steps=1)
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    f = np.float32(W.random_fields(n, 8)[1])
    src = torch.empty(ncell, dtype=torch.float32, pin_memory=True)
    dst = torch.full((ncell + 64,), -7.0, dtype=torch.float32, pin_memory=True)
    src.numpy()[:] = f.ravel()
    ptr = lambda t: C.cast(t.data_ptr(), C.POINTER(C.c_float))
    fdtd._check(fdtd.lib().fdtd_write_field(plan.h, 1, ptr(src), st))
    src.zero_()  # the copy is done when the call returns
    fdtd._check(fdtd.lib().fdtd_read_field(plan.h, 1, ptr(dst), st))
    assert np.array_equal(dst.numpy()[:ncell], f.ravel())
    assert np.all(dst.numpy()[ncell:] == -7.0)
    assert np.array_equal(plan.field(1), f)
    plan.close()
