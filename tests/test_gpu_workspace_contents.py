"""What a workspace held before a call does not show in its results: K's padding
is written by every split, the padding rows of M and N are not, and feed only
entries that are never stored.  Calls on a workspace of FP16 NaNs give the bits
(and the range report) of the same calls on zeros."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import log, to_dev

pytestmark = pytest.mark.gpu

# Small tiles, the 256-wide kernels on planes, and those that split A themselves
# (elementwise and termwise at K = 320), all ragged in M and N.
SHAPES = [(300, 200, 100), (1001, 1501, 333), (3100, 4083, 200), (8100, 1900, 320)]


@pytest.mark.parametrize("order", ["elementwise", "termwise", "elementwise_cross_first"])
@pytest.mark.parametrize("overflow", [False, True], ids=["scaled", "range"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_results_do_not_depend_on_what_the_workspace_held(gpu, shape, order, overflow):
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = shape
    A, B = workloads.make_operands(M, N, K, M + K, "normal")
    if overflow:
        B[K - 1, N - 1] = np.float32(40.0)
    log(f"workspace contents {M}x{N}x{K} {order} overflow={overflow}")
    dA, dB = to_dev(A), to_dev(B)
    code = binding.ORDERS[order]
    stream = torch.cuda.current_stream().cuda_stream

    def results(byte):
        out = []

        def call(what):
            ws = torch.full((n,), byte, dtype=torch.uint8, device="cuda")
            C = torch.full((M, N), float("nan"), device="cuda")
            st = what(C, ws)
            assert st == 0, binding.sgemm_cube_status_string(st)
            assert bool(torch.isfinite(C).all())
            out.append(C.view(torch.int32))

        def compute_a(C, ws):
            assert binding.sgemm_cube_prepare(M, N, K, None, K, dB.data_ptr(), N, 2048.0,
                                              ws.data_ptr(), n, stream) == 0
            return binding.sgemm_cube_compute_a(M, N, K, dA.data_ptr(), K, C.data_ptr(), N, 2048.0,
                                                code, ws.data_ptr(), n, stream)

        n = binding.sgemm_cube_workspace_size(M, N, K)
        call(lambda C, ws: binding.sgemm_cube_ws(M, N, K, dA.data_ptr(), K, dB.data_ptr(), N,
                                                 C.data_ptr(), N, 2048.0, code, ws.data_ptr(), n,
                                                 stream))
        call(compute_a)
        for options in (0, binding.OPT_PRESCALE):
            n = binding.sgemm_cube_ex_workspace_size(M, N, K, code, options)
            bits = torch.full((1,), -1, dtype=torch.int32, device="cuda")
            call(lambda C, ws: binding.sgemm_cube_ex(M, N, K, dA.data_ptr(), K, dB.data_ptr(), N,
                                                     C.data_ptr(), N, 2048.0, code, options,
                                                     ws.data_ptr(), n, bits.data_ptr(), stream))
            out.append(bits)
        return out

    for zeros, nans in zip(results(0), results(0x7E)):
        assert torch.equal(zeros, nans)
