"""Where dense parameters and results pass (needs an MI355X): through pinned
memory up to N = 254 and through a device buffer beyond, straight from and to
the caller's device arrays, and through the buffer for those that a kernel may
not use in place (not on an 8-byte boundary, pinned host memory passed as
device memory).  Every way has to give the same bits.
"""
import ctypes

import numpy as np
import pytest

from oracle import glm_oracle as O
from parity_check import check
from test_gpu_recurrence import TOL, params
from test_gpu_spikes import DT, raster

pytestmark = pytest.mark.gpu


def arrays(kind, sizes):
    """Arrays of float64 of the given sizes: their addresses, and a function that reads one."""
    import torch
    keep = []
    for n in sizes:
        if kind == "host":
            keep.append(np.zeros(n))
        elif kind == "pinned":
            keep.append(torch.zeros(n, dtype=torch.float64, pin_memory=True))
        else:  # "device", and 4 bytes off
            keep.append(torch.zeros(8 * n + 8, dtype=torch.uint8, device="cuda"))
    off = 4 if kind == "misaligned" else 0
    address = [a.ctypes.data if kind == "host" else a.data_ptr() + off for a in keep]

    def read(k):
        a = keep[k]
        if kind in ("host", "pinned"):
            return np.array(a if kind == "host" else a.numpy())
        return a[off:off + 8 * sizes[k]].cpu().numpy().copy().view(np.float64)

    def write(k, v):
        a = keep[k]
        if kind == "host":
            a[:] = v.ravel()
        elif kind == "pinned":
            a.copy_(torch.from_numpy(v.ravel().copy()))
        else:
            a[off:off + 8 * sizes[k]] = torch.from_numpy(np.ascontiguousarray(v).ravel().view(np.uint8).copy()).cuda()
        torch.cuda.synchronize()
    return address, read, write


@pytest.mark.parametrize("N", [3, 254, 255])
@pytest.mark.parametrize("precision", ["fp64", "bf16"])
def test_every_way_gives_the_same(N, precision):
    import torch
    torch.cuda.init()  # before the library's first call
    import paper_1502_04993_amd as G
    lib = G.L.load()
    B = 2000
    bins, neu = raster(N, B, 0.01, N)
    J, mu = params(N, N)
    c = G.Context(N, B, DT, precision=precision)
    c.set_spikes(bins, neu)
    c.set_kernel(0.01)
    p = ctypes.c_void_p
    ref = None
    for kind in ("host", "device", "misaligned", "pinned"):
        where = G.GLMR_HOST if kind == "host" else G.GLMR_DEVICE
        address, read, write = arrays(kind, [N * N, N])
        write(0, J)
        write(1, mu)
        assert lib.glmr_set_params(c.handle, p(address[0]), p(address[1]), where) == 0
        back, read_back, _ = arrays(kind, [N * N, N])
        assert lib.glmr_get_params(c.handle, p(back[0]), p(back[1]), None, where) == 0
        assert np.array_equal(read_back(0), J.ravel()) and np.array_equal(read_back(1), mu)
        out, read_out, _ = arrays(kind, [N, N * N, N])
        ll = ctypes.c_double()
        assert lib.glmr_eval(c.handle, ctypes.byref(ll), p(out[0]), p(out[1]), p(out[2]), None, where) == 0
        got = dict(ll=ll.value, ll_rows=read_out(0), gJ=read_out(1).reshape(N, N), gmu=read_out(2))
        if ref is None:
            ref = got
        for k, v in got.items():
            assert np.array_equal(v, ref[k]), (kind, k)
    c.close()
    if precision == "fp64":
        check(f"arrays N={N}", ref, O.loglik(bins, neu, N, B, DT, 0.01, J, mu), TOL["fp64"])
