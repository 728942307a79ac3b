"""State transfer and the default stream: a solver on a stream of its own reads and overwrites a caller's device
memory only after the work that was enqueued on it before."""
import ctypes

import pytest

import torch

from paper_1601_08145_amd import inputs as I
from paper_1601_08145_amd import lxw as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True])
def test_earlier_work_on_the_callers_memory(batch):
    mesh = L.Mesh.cart(12, 10, 0.0, 1.0, 0.0, 1.0, [1, 1, 1, 1])
    side = torch.cuda.Stream()
    S = L.Batch([mesh], stream=side) if batch else L.Solver(mesh, stream=side)
    ptr = lambda x: ctypes.c_void_p(x.data_ptr())

    def put(q):  # a batch's device states go through the C interface
        if batch:
            assert L.lib().lxw_batch_set_state(S.h, 0, ptr(q), 0.0, L.DEVICE_PTR) == 0
        else:
            S.set_state(q)

    def get(out):
        if batch:
            assert L.lib().lxw_batch_get_state(S.h, 0, ptr(out), None, L.DEVICE_PTR) == 0
        else:
            S.get_state(out)

    Q = torch.from_numpy(I.random_modal_state(mesh.N, 2, 9, 1)).cuda()
    put(Q)
    a = torch.randn(4096, 4096, device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)  # the library's first call loads code
    torch.cuda.synchronize()

    def work():  # tens of milliseconds on the default stream
        for _ in range(30):
            torch.mm(a, a, out=b)

    old = torch.full_like(Q, 7.0)
    buf, kept = old.clone(), torch.empty_like(old)
    torch.cuda.synchronize()
    work()
    kept.copy_(buf)  # reads the buffer after that work
    get(buf)  # then the state overwrites it
    torch.cuda.synchronize()
    assert torch.equal(kept, old) and torch.equal(buf, Q)

    new = 1.5 * Q
    work()
    buf.copy_(new)  # written after that work
    put(buf)  # then taken as the state
    out = torch.empty_like(Q)
    get(out)
    assert torch.equal(out, new)
