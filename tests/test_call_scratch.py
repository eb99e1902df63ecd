"""Where a call's own scratch memory (w4a16_scratch_bytes) comes from, and the calls that do without it."""
import contextlib
import ctypes

import numpy as np
import pytest

from oracle import w4a16_oracle as orc
from paper_2601_16536_amd import workloads as wl

M, K, N = 400, 4096, 7168  # in tiles of 128 x 256 with a split of the last ones: 29 MB of partials; unsplit it needs nothing


class Block:
    """A block of the current device's memory, on a machine without a device."""

    class device:
        index = 0

    def __init__(self, size):
        self.size = size

    def data_ptr(self):
        return 1 << 20


def empty(size, dtype=None, device=None):
    assert device == "cuda"  # the current device, whose current stream the call runs on: not the device of a tensor
    return Block(size)


@pytest.fixture()
def binding():
    from paper_2601_16536_amd import binding as b
    b.lib()
    assert b.lib().w4a16_scratch_bytes(M, N, K, 128, 0) > 0
    return b


def snapshot_with(pool):
    return lambda *a, **k: [{"device": 0, "address": 0, "total_size": 1 << 19, "segment_pool_id": (0, 0)},
                            {"device": 1, "address": 1 << 19, "total_size": 1 << 21, "segment_pool_id": (0, 0)},
                            {"device": 0, "address": 1 << 19, "total_size": 1 << 21, "segment_pool_id": pool}]


def no_snapshot(*a, **k):
    raise RuntimeError("this allocator keeps no record")


@pytest.mark.parametrize("capturing,snapshot,scratch", [
    (False, no_snapshot, True),             # no capture: the block is the call's until the stream is done with it
    (True, snapshot_with((3, 0)), True),    # a graph that torch records: a pool of its own
    (True, snapshot_with((0, 0)), False),   # a capture torch knows nothing of: the common pool
    (True, no_snapshot, False)])
def test_scratch_under_a_capture_comes_from_the_graphs_own_pool(binding, monkeypatch, capturing, snapshot, scratch):
    import torch
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing)
    monkeypatch.setattr(torch.cuda, "memory_snapshot", snapshot)
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(binding, "_capture_id", lambda: 0)
    assert (binding._scratch(128, M, N, K, 0) is not None) == scratch


def test_the_answer_for_one_capture_is_not_the_next_ones(binding, monkeypatch):
    import torch
    asked = []

    def snapshot(pool):
        record = snapshot_with(pool)
        return lambda: asked.append(pool) or record()

    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    monkeypatch.setattr(torch, "empty", empty)
    for number, pool in ((11, (3, 0)), (12, (0, 0)), (13, (4, 0))):
        monkeypatch.setattr(binding, "_capture_id", lambda: number)
        monkeypatch.setattr(torch.cuda, "memory_snapshot", snapshot(pool))
        for _ in range(3):
            assert (binding._scratch(128, M, N, K, 0) is not None) == (pool != (0, 0))
    assert asked == [(3, 0), (0, 0), (4, 0)]  # once per capture


def test_a_full_device_is_no_error_of_a_call_that_can_do_without(binding, monkeypatch):
    import torch

    def full(*a, **k):
        raise torch.OutOfMemoryError("no room")

    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(torch, "empty", full)
    assert binding._scratch(128, M, N, K, 0) is None


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2601_16536_amd import binding
    assert torch.cuda.is_available()
    X, Wp, s, Zp = wl.make(M, K, N, index=9450)
    rows = [0, 127, 128, 399]
    return torch, binding, binding.to_device(X, Wp, s, Zp), rows, orc.gemm(np.ascontiguousarray(X[rows]), Wp, s, Zp, 128)


def check(Y, rows, ref):
    got = Y.double().cpu().numpy()[rows]
    assert np.max(np.abs(got - ref) / (1e-2 * (1.0 + np.abs(ref)))) <= 1.0


def hip_runtime():
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    hip, vp = ctypes.CDLL(path), ctypes.c_void_p
    hip.hipStreamBeginCapture.argtypes = [vp, ctypes.c_int]
    hip.hipStreamEndCapture.argtypes = [vp, ctypes.POINTER(vp)]
    hip.hipGraphInstantiate.argtypes = [ctypes.POINTER(vp), vp, vp, vp, ctypes.c_size_t]
    hip.hipGraphLaunch.argtypes = [vp, vp]
    hip.hipGraphExecDestroy.argtypes = [vp]
    hip.hipGraphDestroy.argtypes = [vp]
    return hip


@contextlib.contextmanager
def captured_by_hip(torch, stream, launch):
    """Captures on `stream` through the HIP runtime alone; launch[0] then replays."""
    hip, graph, run = hip_runtime(), ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(stream.cuda_stream, 0) == 0
    try:
        yield
    finally:
        rc = hip.hipStreamEndCapture(stream.cuda_stream, ctypes.byref(graph))
    assert rc == 0 and hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, 0) == 0
    launch.append(lambda: hip.hipGraphLaunch(run, stream.cuda_stream))
    launch.append(lambda: (hip.hipGraphExecDestroy(run), hip.hipGraphDestroy(graph)))


@pytest.mark.gpu
def test_replays_of_a_capture_begun_through_hip_leave_other_tensors_alone(gpu):
    """What is allocated after the capture keeps its values through replays, and the replays give the eager result."""
    torch, binding, args, rows, ref = gpu
    stream = torch.cuda.Stream()
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    with torch.cuda.stream(stream):
        torch.empty(1, dtype=torch.uint8, device="cuda")
        kept = torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
        del kept  # a free block that the allocator would hand out for scratch
        torch.cuda.synchronize()
        launch = []
        print("[case] captured through HIP", flush=True)
        with captured_by_hip(torch, stream, launch):
            binding.gemm(*args, 128, out=Y)
        others = [torch.full((n,), 7, dtype=torch.uint8, device="cuda") for n in (32 << 20, 29 << 20, 1 << 20)]
        torch.cuda.synchronize()
        for _ in range(3):
            Y.fill_(float("nan"))
            assert launch[0]() == 0
            torch.cuda.synchronize()
            check(Y, rows, ref)
            assert all(bool((t == 7).all()) for t in others)
        launch[1]()


@pytest.mark.gpu
def test_scratch_of_a_graph_that_torch_records(gpu):
    torch, binding, args, rows, ref = gpu
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    binding.gemm(*args, 128, out=Y)
    eager = Y.clone()
    check(eager, rows, ref)
    graph, seen = torch.cuda.CUDAGraph(), []
    print("[case] captured by torch", flush=True)
    with torch.cuda.graph(graph):
        seen.append(binding._scratch(128, M, N, K, 0) is not None)
        binding.gemm(*args, 128, out=Y)
    assert seen == [True]
    others = [torch.full((n,), 7, dtype=torch.uint8, device="cuda") for n in (32 << 20, 29 << 20)]
    for _ in range(3):
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, eager) and all(bool((t == 7).all()) for t in others)


@pytest.mark.gpu
def test_a_capture_after_calls_that_brought_their_scratch(gpu):
    """M = 64, K = 16384, N = 4096: slices, and every plan that has some needs a buffer.  A call through the binding brings its
    own and leaves the library without; the same shape under a capture, which may not allocate, and with an explicit stream,
    which brings none, then runs unsplit."""
    torch, binding, _, _, _ = gpu
    m, k, n = 64, 16384, 4096
    assert binding.lib().w4a16_scratch_bytes(m, n, k, 128, 0) > 0
    X, Wp, s, Zp = wl.make(m, k, n, index=9460)
    rows = [0, 31, 32, 63]
    ref = orc.gemm(np.ascontiguousarray(X[rows]), Wp, s, Zp, 128)
    args = binding.to_device(X, Wp, s, Zp)
    binding.shutdown()  # the library holds no split buffers now
    Y = torch.empty((m, n), dtype=torch.float16, device="cuda")
    check(binding.gemm(*args, 128), rows, ref)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    print("[case] explicit stream under capture, no buffers", flush=True)
    with torch.cuda.graph(graph):
        binding.gemm(*args, 128, out=Y, stream=torch.cuda.current_stream())
    for _ in range(3):
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        check(Y, rows, ref)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("m,k,n,written", [(64, 16384, 4096, True),   # every split plan needs a buffer: the registered one
                                           (M, K, N, False)])         # has a plan that needs none: calls may overlap
def test_calls_take_no_memory_beside_a_registered_workspace(gpu, m, k, n, written, dtype):
    torch, binding, _, _, _ = gpu
    X, Wp, s, Zp = wl.make(m, k, n, index=9470)
    bf16 = dtype == "bf16"
    if bf16:
        X = wl.make_x_bf16(m, k, index=9470)
    rows = [0, m // 2, m - 1]
    ref = (orc.gemm_bf16 if bf16 else orc.gemm)(np.ascontiguousarray(X[rows]), Wp, s, Zp, 128)
    _, dW, dS, dZ = binding.to_device(np.zeros((1, k), np.float16), Wp, s, Zp)
    dX = torch.from_numpy(X.view(np.int16)).cuda().view(torch.bfloat16) if bf16 else torch.from_numpy(X).cuda()
    gemm = binding.gemm_bf16 if bf16 else binding.gemm
    Y = torch.empty((m, n), dtype=dX.dtype, device="cuda")
    binding.shutdown()
    size = max(binding.workspace_bytes(m, n, k, 128), 4 << 20)
    ws = torch.full((size + 256,), 0x55, dtype=torch.uint8, device="cuda")
    ws = ws[-ws.data_ptr() % 256:][:size]
    torch.cuda.synchronize()
    binding.set_workspace(ws)
    try:
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        print("[case] registered", (m, k, n), dtype, flush=True)
        gemm(dX, dW, dS, dZ, 128, out=Y)
        assert torch.cuda.max_memory_allocated() == before
        check(Y, rows, ref)
        assert bool((ws != 0x55).any()) == written
    finally:
        binding.set_workspace(None)


@pytest.mark.gpu
def test_a_workspace_of_the_shapes_size_is_enough_for_both_formats(gpu):
    """w4a16_workspace_bytes does not ask for the format.  M = 101, K = 12544, N = 3216: FP16's plan needs nothing, BF16's
    best one the partials of its slices; with a registered workspace of that size the BF16 call runs a plan that fits."""
    torch, binding, _, _, _ = gpu
    m, k, n = 101, 12544, 3216
    size = binding.workspace_bytes(m, n, k, 128)
    assert binding.query_plan(m, n, k, 128, bf16=True)["workspace_bytes"] > size >= binding.query_plan(m, n, k, 128)["workspace_bytes"]
    _, Wp, s, Zp = wl.make(1, k, n, index=9480)
    Xb = wl.make_x_bf16(m, k, index=9480)
    rows = [0, 31, 63, 64, 100]
    ref = orc.gemm_bf16(np.ascontiguousarray(Xb[rows]), Wp, s, Zp, 128)
    _, dW, dS, dZ = binding.to_device(np.zeros((1, k), np.float16), Wp, s, Zp)
    dX = torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16)
    ws = torch.full((size + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    ws = ws[-ws.data_ptr() % 256:][:size]
    binding.set_workspace(ws)
    try:
        print("[case] bf16 in a registered workspace", flush=True)
        check(binding.gemm_bf16(dX, dW, dS, dZ, 128), rows, ref)
    finally:
        binding.set_workspace(None)
    print("[case] bf16 with its own scratch", flush=True)
    check(binding.gemm_bf16(dX, dW, dS, dZ, 128), rows, ref)
