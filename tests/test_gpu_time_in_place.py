"""Time domain in place, through the C ABI: an output that begins where an input does, inside it, or just past it, gives what
separate buffers give, with the workspace that the size queries ask for."""
import ctypes as C

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _workspace(torch, et, query, *args):
    n = C.c_size_t()
    assert getattr(et.lib(), query)(*args, C.byref(n)) == 0
    return torch.empty(n.value, dtype=torch.uint8, device="cuda")


def _p(t, at=0):
    return C.c_void_p(t.data_ptr() + 4 * at)


@pytest.mark.parametrize("M,F,n_t", [(1, 16, 16), (3, 300, 512), (5, 300, 4096), (4, 3000, 16384), (2, 20000, 32768), (2, 20000, 65536),
                                      (3000, 300, 4096)])
def test_impulse_response_in_place(et, M, F, n_t):
    import torch
    ctx, g = et.Context(0), W.rng(F + n_t)
    H = torch.as_tensor(g.normal(size=2 * M * F).astype(np.float32)).cuda()
    ws = _workspace(torch, et, "et_impulse_response_workspace_size", M, n_t)
    ref = torch.empty(M * n_t, device="cuda")

    def call(x, y):
        ctx.call("et_impulse_response", M, F, 20e3, 100e3, 1, x, n_t, _p(ws), ws.numel(), y, None)
    call(_p(H), _p(ref))
    room = torch.zeros(4 * M * n_t + 4 * M * F + 64, device="cuda")
    for src, dst in ((0, 0), (M * n_t - 1, 0), (0, M * F), (0, 2 * M * F - 1), (0, 2 * M * F), (M * n_t, 0)):
        room.zero_()
        room[src:src + 2 * M * F] = H
        call(_p(room, src), _p(room, dst))
        e = torch.linalg.norm(room[dst:dst + M * n_t] - ref) / torch.linalg.norm(ref)
        assert float(e) <= 1e-6, (src, dst)   # (two transforms of 2^16 points at most, 16 roundings deep each)


@pytest.mark.parametrize("M,n_t,L", [(1, 64, 1), (3, 1024, 40), (4, 16384, 640), (2, 8192, 4096), (2, 8192, 4097), (3000, 1024, 40)])
def test_receiver_signal_in_place(et, M, n_t, L):
    import torch
    ctx, g = et.Context(0), W.rng(n_t + L)
    n = M * (n_t + L - 1)
    h = torch.as_tensor(g.normal(size=M * n_t).astype(np.float32)).cuda()
    call = torch.as_tensor(g.normal(size=L).astype(np.float32)).cuda()
    ws = _workspace(torch, et, "et_receiver_signal_workspace_size", M, n_t, L)
    ref = torch.empty(n, device="cuda")

    def run(x, s, y):
        ctx.call("et_receiver_signal", M, n_t, x, L, s, 2e-6, _p(ws), ws.numel(), y)
    run(_p(h), _p(call), _p(ref))
    room = torch.zeros(2 * n + 2 * M * n_t + 64, device="cuda")
    for src, dst in ((0, 0), (n - 1, 0), (0, M * n_t - 1), (0, M * n_t), (n, 0)):
        room.zero_()
        room[src:src + M * n_t] = h
        run(_p(room, src), _p(call), _p(room, dst))
        assert float(torch.linalg.norm(room[dst:dst + n] - ref) / torch.linalg.norm(ref)) <= 1e-6, (src, dst)
    for at in (0, n - L):   # the call inside the output
        room.zero_()
        room[at:at + L] = call
        run(_p(h), _p(room, at), _p(room))
        assert float(torch.linalg.norm(room[:n] - ref) / torch.linalg.norm(ref)) <= 1e-6, at
