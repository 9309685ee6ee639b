"""Child process of tests/test_gpu_null_stream.py, so that the library's memory
pool holds nothing but the workspace that the null stream keeps:

    memory   device memory is filled and the null stream has work queued on its
             kept workspace; a call on another stream, whose workspace fits
             only if the kept one is given back, must succeed, and both streams'
             results be those of the first call
    capture  the same while another thread captures a stream: both calls
             succeed, the capture ends well and its graph replays
    capture_blocking
             the same with a blocking stream captured, which the null stream
             synchronises with: there the call cannot wait for the null
             stream, so it is refused with SGEMM_CUBE_ERR_ALLOC and succeeds
             once the capture has ended, which it does well
"""
import os
import sys
import threading

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
ERR_ALLOC = 3
SHAPE = (8192, 8192, 11264)  # a workspace of 704 MiB


def _call(binding, M, N, K, A, B, C, stream):
    return binding.sgemm_cube(M, N, K, A.data_ptr(), K, B.data_ptr(), N, C.data_ptr(), N, 2048.0,
                              binding.TERMWISE, stream)


def _same(torch, X, Y):
    return torch.equal(X.view(torch.int32), Y.view(torch.int32))


def _prepare(torch, binding):
    """Operands, the result of the first null-stream call, which leaves its
    workspace kept, two more results, and memory held so that less than a
    workspace is free."""
    from tests.test_gpu_alloc import _fill_device_memory

    M, N, K = SHAPE
    need = binding.sgemm_cube_workspace_size(M, N, K)
    assert need <= 1 << 30
    A = torch.rand((M, K), device="cuda") - 0.5
    B = torch.rand((K, N), device="cuda") - 0.5
    ref, C0, C1 = (torch.full((M, N), float("nan"), device="cuda") for _ in range(3))
    assert _call(binding, *SHAPE, A, B, ref, 0) == 0
    torch.cuda.synchronize()
    held = _fill_device_memory(torch, need // 2)
    free, _ = torch.cuda.mem_get_info()
    print(f"free {free}, workspace {need}", flush=True)
    assert free < need
    return A, B, ref, C0, C1, held


def memory():
    import torch

    from paper_2507_23387_amd import binding

    A, B, ref, C0, C1, held = _prepare(torch, binding)
    side = torch.cuda.Stream()
    for _ in range(4):
        assert _call(binding, *SHAPE, A, B, C0, 0) == 0
    st = _call(binding, *SHAPE, A, B, C1, side.cuda_stream)
    assert st == 0, binding.sgemm_cube_status_string(st)
    torch.cuda.synchronize()
    assert _same(torch, C0, ref) and _same(torch, C1, ref)
    # And the null stream again, whose kept workspace is gone.
    del held
    torch.cuda.empty_cache()
    C0.fill_(float("nan"))
    assert _call(binding, *SHAPE, A, B, C0, 0) == 0
    torch.cuda.synchronize()
    assert _same(torch, C0, ref)


def _blocking_stream(torch):
    """A stream that synchronises with the null stream (torch's own do not)."""
    import ctypes

    hip = ctypes.CDLL("libamdhip64.so")
    s = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(s), ctypes.c_uint(0)) == 0
    return torch.cuda.ExternalStream(s.value)


def capture(blocking=False):
    import torch

    from paper_2507_23387_amd import binding

    x, y = torch.arange(1000.0, device="cuda"), torch.zeros(1000, device="cuda")
    A, B, ref, C0, C1, held = _prepare(torch, binding)
    side = torch.cuda.Stream()
    cap = _blocking_stream(torch) if blocking else torch.cuda.Stream()
    torch.cuda.synchronize()
    status = []

    def other_thread():
        torch.cuda.set_device(0)
        # Work on the null stream would join a blocking stream's capture.
        for C, stream in ([] if blocking else [(C0, 0)]) + [(C1, side.cuda_stream)]:
            status.append(_call(binding, *SHAPE, A, B, C, stream))
            print("status", status[-1], flush=True)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=cap):
        torch.add(x, 1.0, out=y)
        t = threading.Thread(target=other_thread)
        t.start()
        t.join()
        torch.mul(y, 2.0, out=y)
    torch.cuda.synchronize()
    if blocking:
        assert status == [ERR_ALLOC], status
        assert bool(torch.isnan(C1).all())
    else:
        assert status == [0, 0], status
        assert _same(torch, C0, ref) and _same(torch, C1, ref)
    for rep in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, (x + 1.0) * 2.0), rep
    if blocking:
        assert _call(binding, *SHAPE, A, B, C1, side.cuda_stream) == 0
        torch.cuda.synchronize()
        assert _same(torch, C1, ref)
    del held


if __name__ == "__main__":
    {"memory": memory, "capture": capture,
     "capture_blocking": lambda: capture(True)}[sys.argv[1]]()
    print("ok", flush=True)
