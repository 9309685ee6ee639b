"""The split of both operands in one launch: the planes of one launch for A and
B, of one launch each, and of operands at any 4-byte alignment and leading
dimension are the same bytes (padding included), at sizes around the blocks of
32 rows x 128 k of A and 32 k x 128 n of B.  The tiled planes themselves are
held to the oracle's split by the GEMM tests."""
import pytest

import workloads
from tests.gpu_util import log, padded, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (31, 127, 33), (33, 129, 127), (64, 128, 128), (257, 300, 200)]


@pytest.mark.parametrize("offset,pad", [(0, 4), (1, 1), (3, 2)])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_one_launch_writes_the_planes_of_two(gpu, shape, offset, pad):
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = shape
    A, B = workloads.make_operands(M, N, K, 7 * M + K, "normal")
    log(f"split launch {M}x{N}x{K} offset {offset} pad {pad}")
    stream = torch.cuda.current_stream().cuda_stream
    dA, dB = to_dev(A), to_dev(B)
    _, vA = padded(A, K + pad, offset=offset)
    _, vB = padded(B, N + pad, offset=offset)

    def planes(calls):
        ws = binding.workspace(M, N, K).fill_(0xAB)
        for a, lda, b, ldb in calls:
            assert binding.sgemm_cube_prepare(M, N, K, a, lda, b, ldb, 2048.0, ws.data_ptr(),
                                              ws.numel(), stream) == 0
        torch.cuda.synchronize()
        return ws[256:]  # past the header, whose words hold a stamp per split

    want = planes([(dA.data_ptr(), K, None, N), (None, K, dB.data_ptr(), N)])
    assert torch.equal(want, planes([(dA.data_ptr(), K, dB.data_ptr(), N)]))
    assert torch.equal(want, planes([(vA.data_ptr(), K + pad, vB.data_ptr(), N + pad)]))


@pytest.mark.parametrize("shape", [(256, 4096, 8191), (4096, 256, 8191)],
                         ids=lambda s: "x".join(map(str, s)))
def test_stores_past_the_cache_write_the_same_planes(gpu, shape):
    """Planes of more than 128 MiB (here 136): prepare writes them with
    non-temporal stores, a whole call up to 256 MiB with plain ones.  M and N
    are whole plane rows, so both write every byte past the header."""
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = shape
    assert 128 << 20 < binding.sgemm_cube_workspace_size(M, N, K) < 256 << 20
    A, B = workloads.make_operands(M, N, K, 7 * M + K, "normal")
    log(f"split past the cache {M}x{N}x{K}")
    stream = torch.cuda.current_stream().cuda_stream
    dA, dB = to_dev(A), to_dev(B)
    C = torch.empty((M, N), device="cuda")
    ws = [binding.workspace(M, N, K).fill_(0xAB) for _ in range(2)]
    assert binding.sgemm_cube_prepare(M, N, K, dA.data_ptr(), K, dB.data_ptr(), N, 2048.0,
                                      ws[0].data_ptr(), ws[0].numel(), stream) == 0
    assert binding.sgemm_cube_ws(M, N, K, dA.data_ptr(), K, dB.data_ptr(), N, C.data_ptr(), N,
                                 2048.0, binding.TERMWISE, ws[1].data_ptr(), ws[1].numel(),
                                 stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(ws[0][256:], ws[1][256:])
