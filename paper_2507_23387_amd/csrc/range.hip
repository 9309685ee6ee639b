// Range extensions around the split (the exponent management and overflow
// detection that Sec. 4.2 leaves out of scope and Sec. 7 and 8 list as the way
// to widen the method's range):
//   - power-of-two pre-scaling: the largest finite magnitude of every row of A
//     and every column of B is measured, the splits multiply the row (column)
//     by the power of two that brings it to a fixed exponent, and the product
//     is scaled back entry by entry, C_ij = 2^-(p_i + q_j) C'_ij (exact unless
//     C_ij is FP32-subnormal);
//   - the range report: the OR of the range classes the splits stamped.
#include <type_traits>

#include "internal.h"

namespace sgc {
namespace {

// Four consecutive floats at any 4-byte aligned address (one 16-byte load).
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));

// max(m, |a|), skipping inf and NaN.
__device__ __forceinline__ float max_finite(float m, float a) {
  const float b = __builtin_fabsf(a);
  return b <= 3.4028235e38f ? __builtin_fmaxf(m, b) : m;
}

constexpr int kAbsRows = 4;     // rows of A per workgroup, one per wave
constexpr int kAbsCols = 32;    // columns of B per workgroup: one 128-byte line per row of B
constexpr int kAbsUnroll = 8;   // loads in flight per thread

// Elements c .. c + 3 of a row of n, where n < 4 those there are, then zeros.
__device__ __forceinline__ floatx4_u load_quad(const float* row, int64_t c, int64_t n) {
  if (n >= 4) return *reinterpret_cast<const floatx4_u*>(row + c);
  floatx4_u v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int e = 0; e < 3; ++e)
    if (e < n) v[e] = row[e];
  return v;
}

// First element of the quad that holds element c of a row of n: c, or the row's
// last quad, whose elements before c repeat another lane's.
__device__ __forceinline__ int64_t quad_start(int64_t c, int64_t n) {
  return c + 3 < n ? c : (n >= 4 ? n - 4 : 0);
}

// Largest finite |A[i, :]| of the workgroup's four rows, a wave per row.
__device__ __forceinline__ void absmax_rows(int64_t block, int64_t M, int64_t K,
                                            const float* __restrict__ A, int64_t lda,
                                            uint32_t* __restrict__ row_max) {
  const int lane = threadIdx.x & 63;
  const int64_t i = block * kAbsRows + (threadIdx.x >> 6);
  if (i >= M) return;
  const float* const row = A + i * lda;
  float m = 0.0f;
  // 2048 elements from k0, or those there are (`whole` false).
  auto chunk = [&](int64_t k0, auto whole) {
    const int pieces = whole.value ? kAbsUnroll : static_cast<int>((K - k0 + 255) / 256);
    floatx4_u v[kAbsUnroll];
#pragma unroll
    for (int u = 0; u < kAbsUnroll; ++u) {
      if (u >= pieces) break;
      const int64_t k = k0 + u * 256 + lane * 4;
      if constexpr (whole.value)
        v[u] = *reinterpret_cast<const floatx4_u*>(row + k);
      else
        v[u] = k < K ? load_quad(row, quad_start(k, K), K) : floatx4_u{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int u = 0; u < kAbsUnroll; ++u) {
      if (u >= pieces) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) m = max_finite(m, v[u][e]);
    }
  };
  int64_t k0 = 0;
  for (; k0 + kAbsUnroll * 256 <= K; k0 += kAbsUnroll * 256) chunk(k0, std::true_type{});
  if (k0 < K) chunk(k0, std::false_type{});
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, off));
  if (lane == 0) row_max[i] = __builtin_bit_cast(uint32_t, m);
}

// Largest finite |B[k0 .. k1-1, j]| of 32 columns: thread t takes columns
// 4 (t % 8) .. + 3 of every 32nd row, then the workgroup reduces in LDS.
// kAtomic: raise the maxima (several workgroups per column; non-negative floats
// order like their bit patterns), else store them.  Where N ends inside a quad
// its thread reads the row's last whole quad, eight rows at a time like the
// others (one row at a time, element by element, the others waited for it: a
// pre-scaled termwise call of 3008 x 2043 x 1984 took 153 us, now 121).
template <bool kAtomic>
__device__ __forceinline__ void absmax_cols(int64_t strip, int64_t k0, int64_t k1, int64_t N,
                                            const float* __restrict__ B, int64_t ldb,
                                            uint32_t* __restrict__ col_max) {
  __shared__ float part[32][kAbsCols + 1];
  const int t = threadIdx.x;
  const int64_t j = strip * kAbsCols + (t & 7) * 4;
  float m[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (j < N) {
    const int64_t first = quad_start(j, N);
    // 256 rows from kb, or those there are (`whole` false).
    auto chunk = [&](int64_t kb, auto whole) {
      const int pieces =
          whole.value ? kAbsUnroll : static_cast<int>(min<int64_t>(kAbsUnroll, (k1 - kb + 31) / 32));
      floatx4_u v[kAbsUnroll];
#pragma unroll
      for (int u = 0; u < kAbsUnroll; ++u) {
        if (u >= pieces) break;
        const int64_t k = kb + u * 32 + (t >> 3);
        if constexpr (whole.value)
          v[u] = *reinterpret_cast<const floatx4_u*>(B + k * ldb + first);
        else
          v[u] = k < k1 ? load_quad(B + k * ldb, first, N) : floatx4_u{0.0f, 0.0f, 0.0f, 0.0f};
      }
#pragma unroll
      for (int u = 0; u < kAbsUnroll; ++u) {
        if (u >= pieces) break;
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = max_finite(m[e], v[u][e]);
      }
    };
    int64_t kb = k0;
    if (N >= 4)
      for (; kb + kAbsUnroll * 32 <= k1; kb += kAbsUnroll * 32) chunk(kb, std::true_type{});
    for (; kb < k1; kb += kAbsUnroll * 32) chunk(kb, std::false_type{});
    // Column j + e is element j - first + e of that quad.
    const int shift = static_cast<int>(j - first);
#pragma unroll
    for (int r = 0; r < 3; ++r)
      if (r < shift) {
        m[0] = m[1];
        m[1] = m[2];
        m[2] = m[3];
      }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[t >> 3][(t & 7) * 4 + e] = m[e];
  __syncthreads();
  if (t < kAbsCols && strip * kAbsCols + t < N) {
    float r = part[0][t];
#pragma unroll
    for (int i = 1; i < 32; ++i) r = __builtin_fmaxf(r, part[i][t]);
    uint32_t* const out = col_max + strip * kAbsCols + t;
    if constexpr (kAtomic) {
      if (r > 0.0f) atomicMax(out, __builtin_bit_cast(uint32_t, r));
    } else {
      *out = __builtin_bit_cast(uint32_t, r);
    }
  }
}

// Row maxima of A (the first row_blocks workgroups) and column maxima of B.  A
// column's workgroup walks all of K: 1024^3 5 us in this one launch, against 4 +
// 18.5 us as two, with scalar loads and 64 rows of a column per workgroup.
__global__ __launch_bounds__(256) void absmax_kernel(uint32_t row_blocks, int64_t M, int64_t N,
                                                     int64_t K, const float* __restrict__ A,
                                                     int64_t lda, const float* __restrict__ B,
                                                     int64_t ldb, uint32_t* __restrict__ row_max,
                                                     uint32_t* __restrict__ col_max) {
  if (blockIdx.x < row_blocks)
    absmax_rows(blockIdx.x, M, K, A, lda, row_max);
  else
    absmax_cols<false>(blockIdx.x - row_blocks, 0, K, N, B, ldb, col_max);
}

// Row maxima of A; as a side job the grid clears the column maxima that
// absmax_cols_kernel raises next.
__global__ __launch_bounds__(256) void absmax_rows_kernel(int64_t M, int64_t K,
                                                          const float* __restrict__ A,
                                                          int64_t lda,
                                                          uint32_t* __restrict__ row_max,
                                                          uint32_t* __restrict__ col_max,
                                                          int64_t N) {
  for (int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; j < N;
       j += static_cast<int64_t>(gridDim.x) * 256)
    col_max[j] = 0u;
  for (int64_t b = blockIdx.x; b * kAbsRows < M; b += gridDim.x)
    absmax_rows(b, M, K, A, lda, row_max);
}

// Column maxima of B, kAbsChunk rows of B per workgroup.
constexpr int64_t kAbsChunk = 1024;
__global__ __launch_bounds__(256) void absmax_cols_kernel(int64_t K, int64_t N,
                                                          const float* __restrict__ B,
                                                          int64_t ldb,
                                                          uint32_t* __restrict__ col_max) {
  const int64_t k0 = blockIdx.y * kAbsChunk;
  absmax_cols<true>(blockIdx.x, k0, k0 + kAbsChunk < K ? k0 + kAbsChunk : K, N, B, ldb, col_max);
}

// C_ij := 2^-(p_i + q_j) C_ij, one rounding (ldexp).
__global__ __launch_bounds__(256) void unscale_kernel(int64_t M, int64_t N, float* __restrict__ C,
                                                      int64_t ldc,
                                                      const uint32_t* __restrict__ row_max,
                                                      const uint32_t* __restrict__ col_max,
                                                      int exp_a, int exp_b) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (j >= N) return;
  const int q = prescale_shift(col_max[j], exp_b);
  for (int64_t i = blockIdx.y; i < M; i += gridDim.y) {
    const int p = prescale_shift(row_max[i], exp_a);
    C[i * ldc + j] = __builtin_ldexpf(C[i * ldc + j], -(p + q));
  }
}

// *out = OR of the range classes stamped by the last split of each operand.
__global__ void range_report_kernel(const uint32_t* __restrict__ range, int empty,
                                    uint32_t* __restrict__ out) {
  *out = empty ? 0u : range_report_bits(range);
}

inline unsigned grid_y(int64_t rows) {
  return static_cast<unsigned>(rows < 65535 ? (rows > 0 ? rows : 1) : 65535);
}

}  // namespace

hipError_t launch_absmax(const Planes& p, int64_t M, int64_t N, int64_t K, const float* A,
                         int64_t lda, const float* B, int64_t ldb, hipStream_t stream) {
  const int64_t row_blocks = (M + kAbsRows - 1) / kAbsRows;
  const int64_t strips = (N + kAbsCols - 1) / kAbsCols;
  // One launch while a column's workgroup walks at most 4096 rows (about 12
  // us) and the blocks fit a grid; past that the columns are cut along K, into
  // maxima that a launch before clears.
  if (K <= 4096 && row_blocks + strips <= (1 << 23)) {
    hipLaunchKernelGGL(absmax_kernel, dim3(static_cast<unsigned>(row_blocks + strips)), dim3(256),
                       0, stream, static_cast<uint32_t>(row_blocks), M, N, K, A, lda, B, ldb,
                       p.row_max, p.col_max);
    return hipGetLastError();
  }
  const int64_t rows_grid = row_blocks < (1 << 23) ? row_blocks : (1 << 23);
  hipLaunchKernelGGL(absmax_rows_kernel, dim3(static_cast<unsigned>(rows_grid)), dim3(256), 0,
                     stream, M, K, A, lda, p.row_max, p.col_max, N);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid(static_cast<unsigned>(strips),
                  static_cast<unsigned>((K + kAbsChunk - 1) / kAbsChunk));
  hipLaunchKernelGGL(absmax_cols_kernel, grid, dim3(256), 0, stream, K, N, B, ldb, p.col_max);
  return hipGetLastError();
}

hipError_t launch_unscale(const Planes& p, int64_t M, int64_t N, float* C, int64_t ldc,
                          const RangeOpts& opt, hipStream_t stream) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>((N + 255) / 256), grid_y(M));
  hipLaunchKernelGGL(unscale_kernel, grid, dim3(256), 0, stream, M, N, C, ldc, p.row_max,
                     p.col_max, opt.exp_a, opt.exp_b);
  return hipGetLastError();
}

hipError_t launch_range_report(const Planes& p, bool empty, uint32_t* out, hipStream_t stream) {
  hipLaunchKernelGGL(range_report_kernel, dim3(1), dim3(1), 0, stream, p.range, empty ? 1 : 0,
                     out);
  return hipGetLastError();
}

}  // namespace sgc
