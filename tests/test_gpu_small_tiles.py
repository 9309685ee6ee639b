"""The 32, 64, 128 and 192-wide tile kernels that the library picks for problems
whose 256-wide tiles leave compute units idle, at tile edges and remainders: in
every order (range fallback, s > 2^15, pre-scaling and the report too) bit for
bit the rows and columns of a larger problem that runs on the 256-wide kernels,
whose sampled rows meet the oracle within the bar 2 K 2^-24 |A||B|.  Elementwise
also bit for bit the 256 x 256 sweep kernel on the same planes, termwise the
256 x 128 kernel that splits B itself."""
import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_util import gemm, hgemm, log, to_dev
from tests.helpers import abs_ab, assert_parity, band_rows, read_table

pytestmark = pytest.mark.gpu

# (M, N, K): one 32-wide tile with remainders, grids of 32, 64, 128 and 192-wide
# tiles that end inside a tile (the last past the planes' padded rows: 2600 lies
# in 14 tiles of 192, 2688 rows, and pads to 2816; 2740 in 15, 2880), and the
# 256-wide kernels; K from one step of 64.  The table names each order's tile.
SHAPES = [tuple(int(v) for v in row[:3]) for row in read_table("tile_picks.txt")]
# A problem of these rows and columns runs on the 256-wide kernels in every order
# at every K of SHAPES.
WIDE = (4070, 4090)


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


KINDS = {  # order, scale, B overflows, pre-scaling
    "elementwise": ("elementwise", 2048.0, False, False),
    "elementwise_range": ("elementwise", 2048.0, True, False),
    "elementwise_large_scale": ("elementwise", 65536.0, False, False),
    "termwise": ("termwise", 4096.0, False, False),
    "cross": ("elementwise_cross_first", 2048.0, False, False),
    "cross_range": ("elementwise_cross_first", 2048.0, True, False),
    "cross_large_scale": ("elementwise_cross_first", 65536.0, False, False),
    "hgemm": ("hi_only", 2048.0, False, False),
    "prescale_elementwise": ("elementwise", 2048.0, False, True),
    "prescale_termwise": ("termwise", 2048.0, False, True),
    "prescale_cross": ("elementwise_cross_first", 2048.0, False, True),
}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_rows_and_columns_of_a_wide_problem(gpu, shape, kind):
    """An entry of C depends on its row of A and its column of B alone, so C of
    (A, B) is that part of the product of A's rows and B's columns repeated to
    4070 x 4090, which runs on the 256-wide kernels."""
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = shape
    order, scale, overflow, prescale = KINDS[kind]
    A, B = workloads.make_operands(M, N, K, M + K, "normal")
    if overflow:
        B[K - 1, N - 1] = np.float32(40.0)
    if prescale:
        rng = np.random.default_rng(M)
        exp = rng.integers(-28, 20, (M, 1))
        A = np.ldexp(A, exp).astype(np.float32)
        B = np.ldexp(B, rng.integers(-28, 20, (1, N))).astype(np.float32)
        # An FP16-subnormal hi after the scaling to [2^14, 2^15).
        A[M // 2, K // 2] = np.ldexp(1.0, exp[M // 2, 0] - 32)
    log(f"small tiles {kind} {M}x{N}x{K} and wide")
    dA, dB = to_dev(A), to_dev(B)
    wM, wN = max(M, WIDE[0]), max(N, WIDE[1])
    wA = dA[torch.arange(wM, device="cuda") % M].contiguous()
    wB = dB[:, torch.arange(wN, device="cuda") % N].contiguous()

    def call(a, b):
        if order == "hi_only":
            return binding.hgemm(a, b), None
        if prescale:
            return binding.matmul_ex(a, b, scale=scale, order=order, prescale=True, report=True)
        return binding.matmul(a, b, scale=scale, order=order), None

    C, bits = call(dA, dB)
    W, wbits = call(wA, wB)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(C).all())
    assert torch.equal(C.view(torch.int32), W[:M, :N].contiguous().view(torch.int32))
    rows = band_rows(wM, K)
    Ah, Wh = A[rows % M], W.cpu().numpy()[rows]
    Bw = wB.cpu().numpy()
    if prescale:
        assert int(bits.item()) == int(wbits.item()) == binding.RANGE_HI_SUBNORMAL
        # A line's power of two follows from the line, so sampled rows suffice.
        want = oracle.sgemm_prescaled(Ah, Bw, scale, order, kb=32)
    else:
        want = oracle.sgemm(Ah, Bw, scale, order, kb=32)
    assert_parity(Wh, want, K, abs_ab(Ah, Bw), f"wide {kind} {shape}")


@pytest.mark.parametrize("shape", [(298, 8200, 512), (190, 9001, 1000), (700, 30000, 192)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("order", ["elementwise", "termwise", "elementwise_cross_first", "hi_only"])
def test_grids_of_consecutive_tiles_per_xcd(gpu, shape, order):
    """A few rows of tiles against a B of more than 16 MiB, whose tiles are dealt
    out to the XCDs in runs (grids that are no multiple of 8): bit for bit the
    products with parts of B, which are below that size."""
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = shape
    A, B = workloads.make_operands(M, N, K, M + K, "normal")
    log(f"tiles per XCD {order} {M}x{N}x{K}")
    dA, dB = to_dev(A), to_dev(B)

    def call(b):
        return binding.hgemm(dA, b) if order == "hi_only" else binding.matmul(dA, b, order=order)

    C = call(dB)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(C).all())
    for j in range(0, N, 2050):
        part = call(dB[:, j:j + 2050].contiguous())
        assert torch.equal(C[:, j:j + 2050].contiguous().view(torch.int32), part.view(torch.int32))


@pytest.mark.parametrize("bit", ["clean", "all"])
def test_report_of_a_wide_problem(gpu, bit):
    """The report without pre-scaling after a 256-wide GEMM: none and all of the
    range classes."""
    import torch

    from paper_2507_23387_amd import binding

    M, N, K = WIDE + (64,)
    A, B = workloads.make_operands(M, N, K, 5, "uniform_pm1")
    A, B = np.sign(A) * (np.abs(A) + 1), np.sign(B) * (np.abs(B) + 1)  # no subnormal hi
    if bit == "all":
        A[M - 1, K - 1], A[7, 3] = 70000.0, 2.0**-20
        B[K - 1, N - 1], B[3, 5] = np.nan, 32784.0
    log(f"report of a wide problem: {bit}")
    C, bits = binding.matmul_ex(to_dev(A), to_dev(B), scale=4096.0, order="termwise", report=True)
    torch.cuda.synchronize()
    want = oracle.range_classes(A, 4096.0) | oracle.range_classes(B, 4096.0)
    assert int(bits.item()) == want == (15 if bit == "all" else 0)


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
