"""Creating a handle beside an error that another call of the thread left pending."""
import ctypes as C

import pytest

import workloads as W
from tests.test_gpu_batch import lbfd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "bf16dev"])
def test_create_leaves_others_errors_alone(lbfd, prec):  # noqa: F811
    import torch

    lib = lbfd.load()
    p, _ = W.droplet_adsorption(n=32, radius=8.0, precision=prec)
    n = lbfd.workspace_bytes(p)
    ws = torch.empty(n + 256, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    lib.hipGetLastError()
    error = lib.hipSetDevice(9999)   # refused by the runtime, and kept as the thread's last error
    assert error != 0
    h = C.c_void_p()
    st = lib.lbfd_create(C.byref(lbfd.params_struct(p)), C.c_void_p((ws.data_ptr() + 255) & ~255), C.c_size_t(n),
                         C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(h))
    pending = lib.hipGetLastError()
    assert st == lbfd.LBFD_OK and h.value
    assert pending == error
    torch.cuda.synchronize()
    lib.lbfd_destroy(h)
