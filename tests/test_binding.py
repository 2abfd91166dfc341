"""When the binding allocates and binds a workspace (on the CPU: the calls are recorded, nothing is launched)."""
import ctypes
import threading
import types

import numpy as np
import pytest
import torch

from paper_2307_05740_amd import binding


@pytest.fixture
def handle(monkeypatch):
    """An ArrowSpMM without a device, and the list of what its workspace handling does."""
    did = []

    def empty(nbytes, dtype, device):
        did.append(("empty", nbytes))
        return torch.empty(nbytes, dtype=dtype)

    stream = types.SimpleNamespace(synchronize=lambda: did.append(("synchronize",)))
    op = binding.ArrowSpMM.__new__(binding.ArrowSpMM)
    op._torch = types.SimpleNamespace(cuda=types.SimpleNamespace(current_stream=lambda device: stream), empty=empty,
                                      uint8=torch.uint8, OutOfMemoryError=torch.OutOfMemoryError)
    op.device, op._ws, op._ws_k = torch.device("cpu"), None, 0
    op.n = 300
    op.h = binding.arrow_decompose(np.arange(301, dtype=np.int64), np.arange(300, dtype=np.int32), np.ones(300, np.float32), 64)
    monkeypatch.setattr(binding, "arrow_set_workspace", lambda h, ptr, nbytes: did.append(("bind", ptr, nbytes)))
    yield op, did
    binding.arrow_destroy(op.h)
    op.h = 0


def test_a_workspace_that_suffices_stays(handle):
    """A captured graph may hold its address, and a call that finds it may be captured itself: no second buffer is
    worth another workspace."""
    op, did = handle
    op._ensure_workspace(24)
    ws = op._ws
    del did[:]
    for k, second in ((24, True), (24, False), (7, True), (1, False)):
        op._ensure_workspace(k, second=second)
    assert did == [] and op._ws is ws


def test_a_second_buffer_is_asked_for_only_where_it_is_used(handle):
    op, did = handle
    extra = []
    for k, second in ((8, True), (16, False), (32, True)):
        op._ensure_workspace(k, second=second)
        extra.append(op._ws.numel() - max(binding.arrow_workspace_bytes(op.h, k), 256))
    assert extra == [-(-300 * 8 * 4 // 256) * 256, 0, -(-300 * 32 * 4 // 256) * 256]


class Dense:
    """What the general way asks of a tensor."""
    is_cuda, dtype = True, torch.float32
    def __init__(self, *shape): self.shape = shape
    def dim(self): return len(self.shape)
    def is_contiguous(self): return True
    def numel(self): return int(np.prod(self.shape))
    def data_ptr(self): return 4096


def test_a_workspace_that_could_not_be_replaced_is_offered_to_no_call(handle, monkeypatch):
    """The old one is given back before the new one is asked for, so a call after that has none, however few columns it
    has: the native call must not be made with the old number of them, but the general way bind a new one."""
    op, did = handle
    offered, room = [], [1 << 40]
    torch_empty = op._torch.empty

    def empty(nbytes, dtype, device):
        if nbytes > room[0]:
            raise torch.OutOfMemoryError
        return torch_empty(nbytes, dtype, device)

    def native(name, most):                        # as in tensor_call.cpp: a call with more columns than `most` is not plain
        def call(*args):
            offered.append((name, args[most], op._ws is not None))
            return 1 if args[-1].shape[-1] <= args[most] else 0
        return call

    op._torch.empty, op._torch.float32 = empty, torch.float32
    op._call = types.SimpleNamespace(spmm=native("spmm", 4), sddmm=lambda *a: native("sddmm", 4)(*a[:-1]))
    op._index, op._nnz, op._map, op.info, op._spmm, op._sddmm = 0, 300, object(), {"nnz": 300}, 0, 0
    monkeypatch.setattr(binding, "_current_stream", lambda torch, device: 0)
    monkeypatch.setattr(binding, "arrow_spmm", lambda h, x, y, k, stream: did.append(("spmm", k)))
    monkeypatch.setattr(binding, "arrow_sddmm", lambda h, u, v, s, k, stream: did.append(("sddmm", k)))
    X, wide, S = Dense(300, 8), Dense(300, 4096), Dense(300)
    for call in (lambda: op.spmm(X, X), lambda: op.sddmm(X, X, S)):
        op._ensure_workspace(8)
        room[0] = 1 << 16
        with pytest.raises(torch.OutOfMemoryError):
            op.spmm(wide, wide)
        room[0] = 1 << 40
        del offered[:], did[:]
        call()
        assert offered[0][1:] == (0, False) and op._ws is not None and op._ws_k == 8
        assert [d[0] for d in did[1:3]] == ["empty", "bind"] and did[-1][1] == 8
        call()
        assert offered[1][1:] == (8, True) and len(did) == 4
        op._ws, op._ws_k = None, 0

    def refused(h, ptr, nbytes):
        raise binding.ArrowError(-1, "refused")

    monkeypatch.setattr(binding, "arrow_set_workspace", refused)
    with pytest.raises(binding.ArrowError):
        op._ensure_workspace(8)
    assert op._ws_k == 0


@pytest.mark.parametrize("free", [1 << 40, 700_000])
@pytest.mark.parametrize("R", [50, 64])
def test_a_workspace_without_room_for_laid_out_factors_will_do(monkeypatch, R, free):
    """The order-3 product asks for the room that the layout of the factors takes at this rank and the ones below it, then
    for the partial vectors alone: short of memory it is slower, not refused."""
    partials, J, K = 40, 1000, 2000
    least = {50: 8192 + 256, 64: 10_240 + 256}[R]
    want = [768_000 + least] if free > 768_000 + least else [768_000 + least, least]
    asked, bound = [], []

    def empty(nbytes, dtype, device):
        asked.append(nbytes)
        if nbytes > free:
            raise torch.OutOfMemoryError
        return torch.empty(nbytes, dtype=dtype)

    def workspace_bytes(h, r):
        up = lambda n: -(-n // 256) * 256
        return up(partials * r * 4) + (0 if r in (1, 2, 4, 8, 16) or r % 32 == 0 else up((J + K) * -(-r // 32) * 32 * 4)) + 256

    monkeypatch.setattr(binding, "csf3_workspace_bytes", workspace_bytes)
    monkeypatch.setattr(binding, "csf3_set_workspace", lambda h, ptr, nbytes: bound.append(nbytes))
    op = binding.Csf3Mttkrp.__new__(binding.Csf3Mttkrp)
    stream = types.SimpleNamespace(synchronize=lambda: None)
    op._torch = types.SimpleNamespace(cuda=types.SimpleNamespace(current_stream=lambda device: stream), empty=empty,
                                      uint8=torch.uint8, OutOfMemoryError=torch.OutOfMemoryError)
    op.device, op._ws, op._ws_R, op.h, op.info = torch.device("cpu"), None, 0, 0, {"partials": partials, "J": J, "K": K}
    monkeypatch.setattr(binding, "csf3_form", lambda h: binding.CSF3_FORM_SUMS_IN_LDS)
    op._bind_workspace(R)
    assert asked == want and bound == want[-1:] and op._ws.numel() == want[-1] and op._ws_R == R
    free = 0
    with pytest.raises(torch.OutOfMemoryError):
        op._bind_workspace(R + 1)


def test_products_that_share_a_workspace_follow_each_other(monkeypatch):
    """A call on another stream than the last one waits for it, unless it is captured or nothing is written to the workspace."""
    waits, now = [], {}

    class Stream:
        def __init__(self, n): self.cuda_stream = n
        def wait_stream(self, other): waits.append((self.cuda_stream, other.cuda_stream))

    def product(h, B, C, A, R, stream):
        assert stream == now["stream"]

    op = binding.Csf3Mttkrp.__new__(binding.Csf3Mttkrp)
    op._torch = types.SimpleNamespace(float32=torch.float32, cuda=types.SimpleNamespace(
        current_stream=lambda device: Stream(now["stream"]), is_current_stream_capturing=lambda: now["captured"]))
    monkeypatch.setattr(binding, "_current_stream", lambda torch, device: now["stream"])
    monkeypatch.setattr(binding, "csf3_mttkrp", product)
    op.device, op.h, op.info, op._ws_R = torch.device("cpu"), 0, {"I": 2, "J": 3, "K": 4}, 8
    op._ws, op._free_R = object(), 0
    op._last, op._last_raw, op._writes_ws, op._lock = Stream(0), 0, True, threading.Lock()

    class Dense:
        is_cuda, dtype = True, torch.float32
        def __init__(self, rows): self.shape = (rows, 5)
        def dim(self): return 2
        def is_contiguous(self): return True
        def data_ptr(self): return 0

    def call(stream, captured=False):
        now.update(stream=stream, captured=captured)
        op.mttkrp(Dense(3), Dense(4), Dense(2))

    for stream in (0, 0, 7, 7, 0):
        call(stream)
    assert waits == [(7, 0), (0, 7)]
    call(9, captured=True)
    call(0)
    assert len(waits) == 2
    op._writes_ws = False
    call(7)
    assert len(waits) == 2


def test_anything_but_plain_tensors_goes_the_general_way():
    """The native calls take tensors on the handle's device only; for everything else they call nothing and say so, and the
    Python methods then assert and allocate as ever.  (What they ask of a tensor there: test_gpu_edges.py.)"""
    from paper_2307_05740_amd import tensor_call
    called = []
    product = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_void_p] * 3, ctypes.c_int, ctypes.c_void_p)(lambda *a: called.append(a) or 0)
    at = ctypes.cast(product, ctypes.c_void_p).value
    X = torch.zeros(4, 8)
    for x in (X, X.double(), X[:, ::2], X[0], torch.nn.Parameter(X), X.to("meta"), X.to_sparse(), X.numpy(), None):
        assert tensor_call.spmm(at, 0, 0, 4, 8, x, X) == 0
        assert tensor_call.sddmm(at, 0, 0, 4, 8, 3, x, X, X) == 0
        assert tensor_call.mttkrp(at, 0, 0, 4, 4, 4, 8, x, X, X) == 0
    assert called == []
    for call in (tensor_call.spmm, tensor_call.sddmm, tensor_call.mttkrp):
        with pytest.raises(TypeError):
            call(at, 0)
        with pytest.raises(TypeError):
            call(*["0"] * {"spmm": 7, "sddmm": 9, "mttkrp": 10}[call.__name__])


@pytest.mark.parametrize("second", [False, True])
@pytest.mark.parametrize("room", ["everything", "the whole workspace", "the least"])
def test_a_workspace_without_room_for_a_head_in_whole_lines_will_do(handle, monkeypatch, second, room):
    """The product asks for a second buffer, then for the workspace with the room for a head in whole lines, then for what it
    cannot do without: short of memory it is slower, not refused."""
    op, did = handle
    k, xy = 31, -(-300 * 31 * 4 // 256) * 256
    scratch = binding.arrow_scratch_bytes(op.h, k)
    monkeypatch.setattr(binding, "arrow_workspace_bytes", lambda h, k: scratch + xy + 19200)
    sizes = [scratch + 2 * xy + 19200] * second + [scratch + xy + 19200, scratch + xy]
    least = {"everything": 0, "the whole workspace": 1 if second else 0, "the least": 2 if second else 1}[room]
    asked, torch_empty = [], op._torch.empty

    def empty(nbytes, dtype, device):
        asked.append(nbytes)
        if nbytes > sizes[least]:
            raise torch.OutOfMemoryError
        return torch_empty(nbytes, dtype, device)

    op._torch.empty = empty
    op._ensure_workspace(k, second=second)
    assert asked == sizes[:least + 1] and op._ws.numel() == sizes[least] and op._ws_k == k
    assert did[-1] == ("bind", op._ws.data_ptr(), sizes[least])
    sizes[least] = 0
    with pytest.raises(torch.OutOfMemoryError):
        op._ensure_workspace(k + 1, second=second)
    assert op._ws_k == 0
