// Split kernels: FP32 -> (FP16 high word, FP16 scaled residual).
//
// Sec. 3.3 and Eq. recover_eqn of arXiv 2507.23387:
//   hi = fl16(a); r = a - hi (exact in FP32); lo = fl16(r * s)
// with fl16 = round to nearest even and gradual underflow.  On gfx950:
//   - v_cvt_f16_f32 rounds with the MODE register's round mode (RNE by
//     default) and keeps FP16 denormals (the kernels are built with the
//     default float_denorm_mode_16_64 = 3, never with flush-to-zero);
//   - the FP32 subtraction keeps FP32 denormals (float_denorm_mode_32 = 3);
//   - the compiler may fuse r * s and the conversion into v_fma_mixlo_f16,
//     which rounds once; r * s is exact because s is a power of two (checked
//     by the C-ABI), so this equals the two-step definition bit for bit.
// All split kernels are HBM-bound elementwise passes: 4 B read and 4 B
// written (hi + lo) per element.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace sgc {
namespace {

// Row-major split.  Thread = 4 consecutive columns of one row; blockIdx.y
// strides over rows.  kVec: X rows are 16-byte aligned and hi/lo rows 8-byte
// aligned, so whole quads move as float4 / 8-byte stores.
template <bool kVec>
__global__ __launch_bounds__(256) void split_rows_kernel(
    int64_t rows, int64_t cols, const float* __restrict__ X, int64_t ldx,
    uint16_t* __restrict__ hi, uint16_t* __restrict__ lo, int64_t ldh, int64_t rows_pad,
    int64_t cols_pad, float s) {
  const int64_t c0 = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) * 4;
  if (c0 >= cols_pad) return;
  for (int64_t i = blockIdx.y; i < rows_pad; i += gridDim.y) {
    float v[4];
    if (kVec && i < rows && c0 + 3 < cols) {
      const float4 f = *reinterpret_cast<const float4*>(X + i * ldx + c0);
      v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (i < rows && c0 + e < cols) ? X[i * ldx + c0 + e] : 0.0f;
    }
    uint16_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split_value(v[e], s, h[e], l[e]);
    uint16_t* hrow = hi + i * ldh + c0;
    uint16_t* lrow = lo + i * ldh + c0;
    if (kVec && c0 + 3 < cols_pad) {
      const uint2 hv = {static_cast<uint32_t>(h[0]) | (static_cast<uint32_t>(h[1]) << 16),
                        static_cast<uint32_t>(h[2]) | (static_cast<uint32_t>(h[3]) << 16)};
      const uint2 lv = {static_cast<uint32_t>(l[0]) | (static_cast<uint32_t>(l[1]) << 16),
                        static_cast<uint32_t>(l[2]) | (static_cast<uint32_t>(l[3]) << 16)};
      *reinterpret_cast<uint2*>(hrow) = hv;
      *reinterpret_cast<uint2*>(lrow) = lv;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c0 + e < cols_pad) {
          hrow[e] = h[e];
          lrow[e] = l[e];
        }
    }
  }
}

// Range classes of one split entry a -> (hi, lo), after any pre-scaling:
//   1  a is inf or NaN
//   2  a is finite but fl16(a) is infinite (|a| >= 65520, Sec. 3.1)
//   4  hi is finite but the scaled residual overflows FP16 (Rule 2, Sec. 4.2)
//   8  hi is a nonzero FP16 subnormal (the 22-bit guarantee of Sec. 4.2 is lost)
__device__ __forceinline__ uint32_t range_class(float a, uint16_t h, uint16_t l) {
  const bool fin = __builtin_isfinite(a);
  const bool h_fin = (h & 0x7c00) != 0x7c00;
  uint32_t c = fin ? 0u : 1u;
  if (fin && !h_fin) c |= 2u;
  if (h_fin && (l & 0x7fff) == 0x7c00) c |= 4u;
  if ((h & 0x7c00) == 0 && (h & 0x03ff) != 0) c |= 8u;
  return c;
}

// Stamp the classes any lane of the wave saw into header words word..word+3
// (one store per class and wave).
__device__ __forceinline__ void report_classes(uint32_t cls, uint32_t* range, int word,
                                               uint32_t stamp) {
#pragma unroll
  for (int b = 0; b < kRangeClasses; ++b) {
    const unsigned long long m = __ballot((cls >> b) & 1u);
    if (m && static_cast<int>(threadIdx.x & 63) == __ffsll(static_cast<long long>(m)) - 1)
      range[word + b] = stamp;
  }
}

// Four consecutive floats at any 4-byte aligned address: one 16-byte load (the
// hardware takes any dword alignment), so rows of any leading dimension are
// read as whole pieces.
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void load8(const float* src, float (&v)[8]) {
  const floatx4_u f0 = *reinterpret_cast<const floatx4_u*>(src);
  const floatx4_u f1 = *reinterpret_cast<const floatx4_u*>(src + 4);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = f0[e];
    v[e + 4] = f1[e];
  }
}

// Both operands of one split launch, cut into blocks of kABlockRows rows x 128
// k of A and 32 k x 128 n of B; the A blocks come first.
constexpr int kABlockRows = 32;
struct SplitArgs {
  float s;
  uint32_t* range;
  int64_t Kp;
  uint32_t a_blocks, blocks;  // of A, of both (32-bit: the kernel divides them)
  // A
  const float* A;
  int64_t lda, M, K;
  uint16_t* a_hi;
  uint16_t* a_lo;
  const uint32_t* row_max;
  int exp_a;
  uint32_t a_stamp;
  // B
  const float* B;
  int64_t ldb, N;
  uint16_t* b_hi;
  uint16_t* b_lo;
  const uint32_t* col_max;
  int exp_b;
  uint32_t b_stamp;
};

// A block of A into the tiled planes: a wave takes 2 x 4 rows x 128 k, lane l 8
// consecutive k of rows l / 16 and l / 16 + 16, so each row is read as one
// 512-byte piece, and the 16-byte chunks a store instruction writes fill 8
// whole 128-byte lines (4 rows x 32 bytes of one tile each).
template <bool kPre, bool kReport, bool kLo, bool kStream>
__device__ __forceinline__ void split_a_block(const SplitArgs& g, uint32_t block) {
  const int lane = threadIdx.x & 63;
  const uint32_t kblocks = static_cast<uint32_t>((g.Kp + 127) / 128);
  const uint32_t rows = block / kblocks;
  const int64_t k0 = static_cast<int64_t>(block - rows * kblocks) * 128 + (lane & 15) * 8;
  const int64_t m0 = static_cast<int64_t>(rows) * kABlockRows + (threadIdx.x >> 6) * 4 + (lane >> 4);
  if (kReport && threadIdx.x == 0) g.range[kWordAStamp] = g.a_stamp;
  if (k0 >= g.Kp) return;
  float v[kABlockRows / 16][8];
#pragma unroll
  for (int u = 0; u < kABlockRows / 16; ++u) {
    const int64_t m = m0 + 16 * u;
    if (m < g.M && k0 + 7 < g.K) {
      load8(g.A + m * g.lda + k0, v[u]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        v[u][e] = (m < g.M && k0 + e < g.K) ? g.A[m * g.lda + k0 + e] : 0.0f;
    }
  }
  uint32_t cls = 0;
#pragma unroll
  for (int u = 0; u < kABlockRows / 16; ++u) {
    const int64_t m = m0 + 16 * u;
    if constexpr (kPre) {
      const int shift = m < g.M ? prescale_shift(g.row_max[m], g.exp_a) : 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[u][e] = __builtin_ldexpf(v[u][e], shift);
    }
    u32x4 hv, lv;
    split8(v[u], g.s, hv, lv);
    if constexpr (kReport) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        cls |= range_class(v[u][2 * e], hv[e] & 0xffff, lv[e] & 0xffff);
        cls |= range_class(v[u][2 * e + 1], hv[e] >> 16, lv[e] >> 16);
      }
    }
    const int64_t idx = tiled_index(m, k0, g.Kp);
    store_chunk<kStream>(g.a_hi + idx, hv);
    if constexpr (kLo) store_chunk<kStream>(g.a_lo + idx, lv);
  }
  if constexpr (kReport) report_classes(cls, g.range, kWordAClass, g.a_stamp);
}

// A block of B into the tiled planes of B transposed (two tiles): thread t
// splits rows k and k+1 (k = 2 (t / 16)) at 8 consecutive n, each wave reading
// eight 512-byte row pieces.  The (k, k+1) pairs of hi and of lo go to LDS as
// 32-bit words, n-major, so each 16-byte chunk of a tile row is one LDS read;
// thread t then writes chunk t of both tiles of both planes (4 KiB contiguous
// per tile).  It also stamps the range flag (see launch_split) when some
// |B_hi| s > 65504, the largest finite FP16 value.
template <bool kPre, bool kReport, bool kLo, bool kStream>
__device__ __forceinline__ void split_b_block(const SplitArgs& g, uint32_t block) {
  constexpr int kK = 2 * kSlice;
  constexpr int kPitch = kK / 2 + 4;  // words per n row; 16-byte aligned rows
  __shared__ __align__(16) uint32_t ph[kPanel * kPitch];
  __shared__ __align__(16) uint32_t pl[kLo ? kPanel * kPitch : 4];
  const int t = threadIdx.x;
  const uint32_t kblocks = static_cast<uint32_t>(g.Kp / kK);
  const int64_t panel = block / kblocks;
  const int64_t kblock = block - static_cast<uint32_t>(panel) * kblocks;
  const int nl = (t & 15) * 8;
  const int kp = t >> 4;  // k pair
  const int64_t k = kblock * kK + 2 * kp;
  const int64_t n = panel * kPanel + nl;
  float v0[8], v1[8];
  if (k + 1 < g.K && n + 7 < g.N) {
    load8(g.B + k * g.ldb + n, v0);
    load8(g.B + (k + 1) * g.ldb + n, v1);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v0[e] = (k < g.K && n + e < g.N) ? g.B[k * g.ldb + n + e] : 0.0f;
      v1[e] = (k + 1 < g.K && n + e < g.N) ? g.B[(k + 1) * g.ldb + n + e] : 0.0f;
    }
  }
  if constexpr (kPre) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int shift = n + e < g.N ? prescale_shift(g.col_max[n + e], g.exp_b) : 0;
      v0[e] = __builtin_ldexpf(v0[e], shift);
      v1[e] = __builtin_ldexpf(v1[e], shift);
    }
  }
  bool big = false;
  uint32_t cls = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    uint16_t h0, l0, h1, l1;
    split_value(v0[e], g.s, h0, l0);
    split_value(v1[e], g.s, h1, l1);
    big |= __builtin_fabsf(static_cast<float>(__builtin_bit_cast(_Float16, h0))) * g.s > 65504.0f;
    big |= __builtin_fabsf(static_cast<float>(__builtin_bit_cast(_Float16, h1))) * g.s > 65504.0f;
    if constexpr (kReport) cls |= range_class(v0[e], h0, l0) | range_class(v1[e], h1, l1);
    ph[(nl + e) * kPitch + kp] = static_cast<uint32_t>(h0) | (static_cast<uint32_t>(h1) << 16);
    if constexpr (kLo)
      pl[(nl + e) * kPitch + kp] = static_cast<uint32_t>(l0) | (static_cast<uint32_t>(l1) << 16);
  }
  if (big) g.range[kWordBOverflow] = g.b_stamp;
  if (t == 0) g.range[kWordBStamp] = g.b_stamp;
  if constexpr (kReport) report_classes(cls, g.range, kWordBClass, g.b_stamp);
  __syncthreads();
  const int r = t >> 1;
  const int c = (t & 1) ^ tile_swizzle(r);  // logical chunk stored at position t & 1
#pragma unroll
  for (int sl = 0; sl < kK / kSlice; ++sl) {
    const int64_t base = (panel * (g.Kp / kSlice) + kblock * (kK / kSlice) + sl) * kTileHalves + t * 8;
    store_chunk<kStream>(g.b_hi + base, *reinterpret_cast<const u32x4*>(ph + r * kPitch + sl * 8 + c * 4));
    if constexpr (kLo)
      store_chunk<kStream>(g.b_lo + base, *reinterpret_cast<const u32x4*>(pl + r * kPitch + sl * 8 + c * 4));
  }
}

// The split of A, of B or of both in one launch.  HBM-bound at size (8192^3: 187
// us for 1 GiB moved, 5.7 TB/s; 192 us as two launches; B's blocks first 197);
// below about 10 MB a launch, 4 us, is all it costs, hence one for both
// operands (256^3: 8.7 to 5.0 us).  2777 x 3001 x 1531, whose rows have no
// 16-byte alignment: 24.2 us with scalar loads in two launches, 12.6 so.
template <bool kPre, bool kReport, bool kLo, bool kStream>
__global__ __launch_bounds__(256) void split_tiled_kernel(SplitArgs g) {
  uint32_t b = blockIdx.x;
  for (; b < g.a_blocks; b += gridDim.x) split_a_block<kPre, kReport, kLo, kStream>(g, b);
  for (; b < g.blocks; b += gridDim.x) {
    split_b_block<kPre, kReport, kLo, kStream>(g, b - g.a_blocks);
    __syncthreads();  // this block's LDS words are read before the next block's are written
  }
}

__global__ __launch_bounds__(256) void zero_kernel(int64_t M, int64_t N, float* __restrict__ C,
                                                   int64_t ldc) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j >= N) return;
  for (int64_t i = blockIdx.y; i < M; i += gridDim.y) C[i * ldc + j] = 0.0f;
}

inline unsigned grid_rows(int64_t rows) {
  return static_cast<unsigned>(rows < 65535 ? (rows > 0 ? rows : 1) : 65535);
}

}  // namespace

hipError_t launch_split_rows(int64_t rows, int64_t cols, const float* X, int64_t ldx,
                             uint16_t* hi, uint16_t* lo, int64_t ldh, float scale,
                             hipStream_t stream) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const int64_t quads = (cols + 3) / 4;
  const dim3 grid(static_cast<unsigned>((quads + 255) / 256), grid_rows(rows));
  const bool vec = (reinterpret_cast<uintptr_t>(X) % 16 == 0) && (ldx % 4 == 0) &&
                   (reinterpret_cast<uintptr_t>(hi) % 8 == 0) &&
                   (reinterpret_cast<uintptr_t>(lo) % 8 == 0) && (ldh % 4 == 0);
  if (vec)
    hipLaunchKernelGGL(split_rows_kernel<true>, grid, dim3(256), 0, stream, rows, cols, X, ldx,
                       hi, lo, ldh, rows, cols, scale);
  else
    hipLaunchKernelGGL(split_rows_kernel<false>, grid, dim3(256), 0, stream, rows, cols, X, ldx,
                       hi, lo, ldh, rows, cols, scale);
  return hipGetLastError();
}

hipError_t launch_split(const Planes& p, int64_t M, int64_t N, int64_t K, const float* A,
                        int64_t lda, const float* B, int64_t ldb, float scale,
                        const RangeOpts& opt, uint32_t a_stamp, uint32_t b_stamp, SplitPlanes what,
                        hipStream_t stream) {
  // Mp and Np are multiples of 256 and Kp of 64 (plan_planes).  Rows of the
  // planes past M and N only feed entries of C that are never stored, so only
  // kSplitPadded, for planes that outlive the call, fills them.
  SplitArgs g{};
  g.s = scale;
  g.range = p.range;
  g.Kp = p.Kp;
  g.K = K;
  const bool padded = what == kSplitPadded;
  int64_t a_rows = 0, b_rows = 0, a_blocks = 0, b_blocks = 0;
  if (B) {
    // A block that sees |B_hi| s > 65504 writes range[kWordBOverflow] = stamp,
    // every block range[kWordBStamp] = stamp, so the two words are equal
    // afterwards exactly when this split found one; a fresh stamp per call
    // makes a reset pass unnecessary.
    g.B = B, g.ldb = ldb, g.N = N;
    g.b_hi = p.b_hi, g.b_lo = p.b_lo;
    g.col_max = p.col_max, g.exp_b = opt.exp_b, g.b_stamp = b_stamp;
    b_rows = padded ? p.Np : round_up(N, kPanel);
    b_blocks = p.Kp / (2 * kSlice) * (b_rows / kPanel);
  }
  if (A) {
    g.A = A, g.lda = lda, g.M = M;
    g.a_hi = p.a_hi, g.a_lo = p.a_lo;
    g.row_max = p.row_max, g.exp_a = opt.exp_a, g.a_stamp = a_stamp;
    a_rows = padded ? p.Mp : round_up(M, kABlockRows);
    a_blocks = (p.Kp + 127) / 128 * (a_rows / kABlockRows);
  }
  // 2^32 blocks are at least 2^43 planes' bytes, more than any device holds.
  const int64_t blocks = a_blocks + b_blocks;
  if (blocks > UINT32_MAX) return hipErrorInvalidValue;
  g.a_blocks = static_cast<uint32_t>(a_blocks);
  g.blocks = static_cast<uint32_t>(blocks);
  // Non-temporal stores for planes that the 256 MiB last-level cache cannot hold
  // until they are read: above 256 MiB where the GEMM follows at once, above 128
  // MiB for planes that outlive the call.  Plain against non-temporal, us: the
  // split of B of 64 x 8192 x 8192 (256 MiB) 107 and 84, of 4096 x 4096 x 12288
  // (192) 82 and 67, of 64 x 8192 x 4096 (128) 46 and 45, but with the call that
  // reads it 81 and 90; whole calls of 64 x 8192 x 8192 (258) 185 and 180, 4096 x
  // 4096 x 8192 (256) 613 and 621, 1024 x 1024 x 16384 (128) 153 and 195, 48 x 4096
  // x 4096 (64) 43 and 53; 8192^3 and 4096 x 4096 x 16384 (512) the same within 1 %.
  // Smaller planes that outlive the call take longer to write plain (2229 problems
  // of 8 to 128 MiB: 6-9 % on average, 2048 x 4096 of B 15 us against 10.5), but
  // with the GEMM that reads them next the two are 7-15 % faster.
  const int64_t bytes = (a_rows + b_rows) * p.Kp * (what == kSplitHigh ? 2 : 4);
  const bool past_cache = bytes > (padded ? int64_t{128} << 20 : int64_t{256} << 20);
  // At most 2^22 workgroups (a grid dimension holds less than 2^32 threads);
  // past that each takes several blocks.
  const dim3 grid(std::min(g.blocks, 1u << 22));
  auto launch = [&](auto pre, auto report, auto lo) {
    if (past_cache)
      hipLaunchKernelGGL((split_tiled_kernel<pre.value, report.value, lo.value, true>), grid,
                         dim3(256), 0, stream, g);
    else
      hipLaunchKernelGGL((split_tiled_kernel<pre.value, report.value, lo.value, false>), grid,
                         dim3(256), 0, stream, g);
  };
  const std::true_type yes;
  const std::false_type no;
  if (what == kSplitHigh)
    launch(no, no, no);
  else if (opt.prescale && opt.report)
    launch(yes, yes, yes);
  else if (opt.prescale)
    launch(yes, no, yes);
  else if (opt.report)
    launch(no, yes, yes);
  else
    launch(no, no, yes);
  return hipGetLastError();
}

hipError_t launch_zero(int64_t M, int64_t N, float* C, int64_t ldc, hipStream_t stream) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>((N + 255) / 256), grid_rows(M));
  hipLaunchKernelGGL(zero_kernel, grid, dim3(256), 0, stream, M, N, C, ldc);
  return hipGetLastError();
}

}  // namespace sgc
