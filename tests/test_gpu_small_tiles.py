"""The 32, 64, 128 and 192-wide tile kernels that the library picks for problems
whose 256-wide tiles leave compute units idle, at tile edges and remainders.

Elementwise: bit for bit the 256 x 256 sweep kernel on the same planes (scaled
body, range fallback, s > 2^15).  Termwise: bit for bit the 256 x 128 kernel
that splits B itself.  Cross-terms-first (both bodies) and the FP16 baseline:
the oracle, within the bar 2 K 2^-24 |A||B|."""
import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_util import gemm, hgemm, log, to_dev
from tests.helpers import abs_ab, assert_parity, band_rows

pytestmark = pytest.mark.gpu

# (M, N, K): one 32-wide tile with remainders, grids of 32, 64, 128 and 192-wide
# tiles that end inside a tile (the last past the planes' padded rows: 2600 lies
# in 14 tiles of 192, 2688 rows, and pads to 2816; 2740 in 15, 2880); K from one
# step of 64.
SHAPES = [(31, 36, 64), (257, 260, 192), (512, 512, 64), (700, 1020, 192), (1500, 1660, 704),
          (2777, 3000, 320)]


@pytest.mark.parametrize("overflow,scale", [(False, 2048.0), (True, 2048.0), (False, 65536.0)],
                         ids=["scaled", "range", "large_scale"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_elementwise_gives_the_wide_kernels_bits(gpu, shape, overflow, scale):
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = shape
    A, B = workloads.make_operands(M, N, K, M + K, "normal")
    if overflow:
        B[K - 1, N - 1] = np.float32(40.0)
    log(f"small tiles elementwise {M}x{N}x{K} overflow={overflow} s={scale}")
    dA, dB = to_dev(A), to_dev(B)
    ws = binding.workspace(M, N, K)
    st = torch.cuda.current_stream().cuda_stream
    assert binding.sgemm_cube_prepare(M, N, K, dA.data_ptr(), K, dB.data_ptr(), N, scale,
                                      ws.data_ptr(), ws.numel(), st) == 0
    C = [torch.full((M, N), float("nan"), device="cuda") for _ in range(3)]
    assert binding.sgemm_cube_compute(M, N, K, C[0].data_ptr(), N, scale, 0, ws.data_ptr(),
                                      ws.numel(), st) == 0
    assert binding.sgemm_cube_compute_tile(M, N, K, C[1].data_ptr(), N, scale, 0, 256, 256, 32, 4,
                                           ws.data_ptr(), ws.numel(), st) == 0
    assert binding.sgemm_cube_ws(M, N, K, dA.data_ptr(), K, dB.data_ptr(), N, C[2].data_ptr(), N,
                                 scale, 0, ws.data_ptr(), ws.numel(), st) == 0
    torch.cuda.synchronize()
    assert bool(torch.isfinite(C[0]).all())
    for other in C[1:]:
        assert torch.equal(C[0].view(torch.int32), other.view(torch.int32))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_termwise_gives_the_wide_kernels_bits(gpu, shape):
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = shape
    A, B = workloads.make_operands(M, N, K, M + K, "normal")
    log(f"small tiles termwise {M}x{N}x{K}")
    dA, dB = to_dev(A), to_dev(B)
    got = binding.matmul(dA, dB, order="termwise")
    wide = binding.matmul_ex(dA, dB, order="termwise", split_b_in_gemm=True)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), wide.view(torch.int32))


@pytest.mark.parametrize("kind", ["cross", "cross_range", "hgemm"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_cross_first_and_baseline_against_the_oracle(gpu, shape, kind):
    M, N, K = shape
    A, B = workloads.make_operands(M, N, K, M + K, "normal")
    if kind == "cross_range":
        B[0, 0] = np.float32(40.0)
    log(f"small tiles {kind} {M}x{N}x{K}")
    C = hgemm(A, B) if kind == "hgemm" else gemm(A, B, 2048.0, "elementwise_cross_first")
    assert np.isfinite(C).all()
    rows = band_rows(M, K, band=16)
    order = "hi_only" if kind == "hgemm" else "elementwise_cross_first"
    want = oracle.sgemm_rows(A, B, rows, 2048.0, order, kb=32)
    assert_parity(C[rows], want, K, abs_ab(A, B, rows), f"small tiles {kind} {shape}")


@pytest.mark.parametrize("order", ["elementwise", "termwise"])
@pytest.mark.parametrize("shape", [(5, 33, 4096), (35, 31, 4097), (70, 300, 9000), (1100, 1030, 80)],
                         ids=lambda s: "x".join(map(str, s)))
def test_prescaled_with_the_report(gpu, shape, order):
    """Pre-scaling and the report around the small tiles: the maxima in one
    launch (K <= 4096) and cut along K, the powers of two taken back out in
    the GEMM's store, on rows and columns from 2^-28 to 2^24 and rows of no
    alignment, against the oracle's pre-scaled product."""
    import torch

    from paper_2507_23387_amd import binding
    from tests.gpu_util import padded

    M, N, K = shape
    rng = np.random.default_rng(M + K)
    A = (rng.uniform(-1, 1, (M, K)) * np.ldexp(1.0, rng.integers(-28, 25, (M, 1)))).astype(np.float32)
    B = (rng.uniform(-1, 1, (K, N)) * np.ldexp(1.0, rng.integers(-28, 25, (1, N)))).astype(np.float32)
    A[M - 1, K - 1] = np.float32(2.0**30)  # the last entry of a row holds its maximum
    log(f"prescale {order} {M}x{N}x{K}")
    _, vA = padded(A, K + 1, offset=1)
    _, vB = padded(B, N + 3, offset=2)
    C, bits = binding.matmul_ex(vA[:, :K], vB[:, :N], order=order, prescale=True, report=True)
    torch.cuda.synchronize()
    rows = band_rows(M, K, band=64)
    want = oracle.sgemm_prescaled(A[rows], B, 2048.0, order, kb=32)
    assert_parity(C.cpu().numpy()[rows], want, K, abs_ab(A, B, rows), f"prescale {shape}")
    # Entries far below their row's largest have subnormal high words, no other class occurs.
    assert int(bits.item()) & ~binding.RANGE_HI_SUBNORMAL == 0
