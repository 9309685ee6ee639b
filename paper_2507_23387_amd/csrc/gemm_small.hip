// Three-product MFMA GEMM on prepared FP16 planes for problems whose 256-wide
// tiles would leave most of the 256 compute units idle (gfx950).
//
// gemm_small_kernel<V, kBM, kBN, kWM, kWN, kStages> computes a kBM x kBN tile
// of C per workgroup of kWM x kWN waves, in every accumulation order and for
// the FP16 baseline.  Per accumulator it applies the MFMAs (and block folds)
// of gemm.hip's kernels in the same order, so its results are theirs bit for
// bit, whatever the tile.
//
// The orders with a range fallback (elementwise, cross-terms-first) have both
// bodies in one kernel: a workgroup reads the range flag and runs the one that
// applies, so these orders take one launch here.
//
// What bounds it: at these sizes a 256 x 256 kernel runs on M N / 65536 compute
// units at 1.6 us per 32-wide k-step.  A smaller tile spreads the same k-steps
// over more compute units but copies and reads more LDS bytes per MFMA: a
// 64 x 64 step reads 48 KiB (8 waves of 16 x 32) and copies 16 KiB through LDS
// for 96 cycles of MFMAs per SIMD and takes 0.24 us, near the 128 B per clock
// of the LDS; a 32 x 32 step takes 0.11 us, the latency of a barrier, an LDS
// read and three dependent MFMAs.  So the tile is the smallest that still
// leaves few workgroups per compute unit.  GEMM alone, elementwise, wide kernel
// against this one: 256^3 25.9 and 4.2 us, 300 x 200 x 1024 60 and 6.5,
// 1024^3 60 and 12.2, 48 x 4096 x 4096 196 and 18, 2048 x 2048 x 2816 142 and
// 65; hgemm at 2048 x 2048 x 2816 91 and 31 us.
#include <algorithm>
#include <atomic>

#include "gemm_common.h"

namespace sgc {
namespace {

// How a tile's products are accumulated (gemm.hip describes each).
enum Fold : int { kElScaled, kElUnscaled, kTermFold, kCrScaled, kCrUnscaled, kHiFold };

constexpr int kSmallStep = 2 * kSlice;  // k per MFMA step and per stage (32)

template <int kBM_, int kBN_, int kWM, int kWN, int kStages_, bool kHi>
struct SmallShape {
  static constexpr int kBM = kBM_, kBN = kBN_, kStages = kStages_;
  static constexpr int kPlanes = kHi ? 1 : 2;
  static constexpr int kWaves = kWM * kWN;
  static constexpr int kWavesN = kWN;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kWRows = kBM / kWM, kWCols = kBN / kWN;  // per wave
  static constexpr int kRT = kWRows / 16, kCT = kWCols / 16;    // 16 x 16 blocks per wave
  // One operand plane of one stage in LDS: slice-major, 32 bytes per row.
  static constexpr int kAPlane = 2 * kBM * kSlice;  // halves
  static constexpr int kBPlane = 2 * kBN * kSlice;
  static constexpr int kBBase = kPlanes * kAPlane;
  static constexpr int kSlot = kBBase + kPlanes * kBPlane;
  static constexpr size_t kLdsBytes = static_cast<size_t>(kStages) * kSlot * 2;
  // 1 KiB copies (32 rows of one slice of one plane) per stage.
  static constexpr int kUnits = kPlanes * 2 * (kBM + kBN) / 32;
  static constexpr int kDma = kUnits / kWaves;  // per wave
  static_assert(kBM % 32 == 0 && kBN % 32 == 0 && kPanel % kBM == 0 && kPanel % kBN == 0,
                "tiles are whole 32-row pieces of one panel");
  static_assert(kWRows % 16 == 0 && kWCols % 16 == 0, "whole MFMA tiles per wave");
  static_assert(kUnits % kWaves == 0, "every wave issues the same number of copies");
  static_assert(kStages >= 3, "the ring holds the stage read, one landing, one in flight");
  static_assert(kLdsBytes <= kMaxLdsBytes, "LDS of every kernel stays within 128 KiB");
};

struct SmallArgs {
  const uint16_t* a_hi;
  const uint16_t* a_lo;
  const uint16_t* b_hi;
  const uint16_t* b_lo;
  const uint32_t* range;
  int Kp, tiles_m, tiles_n;
  float* C;
  int64_t ldc;
  int M, N;
  float s, inv_s;
  // Pre-scaling (row_max not null): C_ij is stored times 2^-(p_i + q_j).
  const uint32_t* row_max;
  const uint32_t* col_max;
  int exp_a, exp_b;
  uint32_t* report;  // range report word, or null
};

template <class S, int kFold>
__device__ __forceinline__ void small_tile(const SmallArgs& g, uint16_t* lds) {
  constexpr int kRT = S::kRT, kCT = S::kCT;
  int tm, tn;
  tile_of<4>(blockIdx.x, g.tiles_m, g.tiles_n, tm, tn);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = w / S::kWavesN, wn = w % S::kWavesN;
  const int ksteps = g.Kp / kSmallStep;

  // Copy u of a stage is 1 KiB: rows 32 r .. 32 r + 31 of one slice of one
  // plane, contiguous in the tiled plane; the A planes come first, and wave w
  // issues copies w, w + kWaves, ...
  constexpr int kAU = S::kPlanes * 2 * S::kBM / 32;
  const int64_t panel_bytes = static_cast<int64_t>(g.Kp) * kPanel * 2;
  const unsigned lds_base = lds_address(lds);
  const char* src[S::kDma];
  unsigned dst[S::kDma];
#pragma unroll
  for (int i = 0; i < S::kDma; ++i) {
    const int u = i * S::kWaves + w;
    const bool is_a = u < kAU;
    const int v = is_a ? u : u - kAU;
    const int per_slice = (is_a ? S::kBM : S::kBN) / 32;
    const int p = v / (2 * per_slice), sl = v / per_slice % 2, r = v % per_slice;
    const int row0 = is_a ? tm * S::kBM : tn * S::kBN;
    const uint16_t* plane = is_a ? (p ? g.a_lo : g.a_hi) : (p ? g.b_lo : g.b_hi);
    src[i] = reinterpret_cast<const char*>(plane) + (row0 / kPanel) * panel_bytes +
             sl * (kTileHalves * 2) + (row0 % kPanel + 32 * r) * (kSlice * 2);
    dst[i] = lds_base + ((is_a ? p * S::kAPlane : S::kBBase + p * S::kBPlane) +
                         (sl * (is_a ? S::kBM : S::kBN) + 32 * r) * kSlice) * 2;
  }
  // Stage t into ring slot `slot`; past the end the last stage again.
  auto copy_one = [&](int t, int slot, int i) {
    const int64_t off = static_cast<int64_t>(min(t, ksteps - 1)) * (2 * kTileHalves * 2);
    dma16s(src[i] + off, lane * 16, dst[i] + slot * (S::kSlot * 2));
  };

  // Fragment of 16-row block i of a plane: row l % 16, k chunk l / 16 of the
  // step, i.e. chunk (l / 16) % 2 of slice l / 32, swapped when bit 4 of the
  // row is set (blocks of odd index, counted from the wave's first row).
  const int fr = lane & 15, fc = lane >> 4;
  const int a_par = S::kWRows % 32 == 0 ? 0 : wm & 1, b_par = S::kWCols % 32 == 0 ? 0 : wn & 1;
  int a_off[2], b_off[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    a_off[x] = ((fc >> 1) * S::kBM + wm * S::kWRows + fr) * kSlice + (((fc & 1) ^ x ^ a_par) << 3);
    b_off[x] = S::kBBase + ((fc >> 1) * S::kBN + wn * S::kWCols + fr) * kSlice +
               (((fc & 1) ^ x ^ b_par) << 3);
  }
  auto rd_a = [&](int slot, int p, int i) -> half8 {
    return *reinterpret_cast<const half8*>(lds + slot * S::kSlot + p * S::kAPlane + a_off[i & 1] +
                                           i * 16 * kSlice);
  };
  auto rd_b = [&](int slot, int p, int j) -> half8 {
    return *reinterpret_cast<const half8*>(lds + slot * S::kSlot + p * S::kBPlane + b_off[j & 1] +
                                           j * 16 * kSlice);
  };
  struct Frags {
    half8 ah[kRT], al[kRT], bh[kCT], bl[kCT];
  };
  auto read = [&](Frags& f, int slot) {
#pragma unroll
    for (int i = 0; i < kRT; ++i) {
      f.ah[i] = rd_a(slot, 0, i);
      if constexpr (kFold != kHiFold) f.al[i] = rd_a(slot, 1, i);
    }
#pragma unroll
    for (int j = 0; j < kCT; ++j) {
      f.bh[j] = rd_b(slot, 0, j);
      if constexpr (kFold != kHiFold) f.bl[j] = rd_b(slot, 1, j);
    }
  };

  const _Float16 s16 = static_cast<_Float16>(g.s);
  const half8 s8 = {s16, s16, s16, s16, s16, s16, s16, s16};
  constexpr bool kTerm = kFold == kTermFold;
  floatx4 acc[kRT][kCT], xa[kTerm ? kRT : 1][kTerm ? kCT : 1], xb[kTerm ? kRT : 1][kTerm ? kCT : 1];
#pragma unroll
  for (int i = 0; i < kRT; ++i)
#pragma unroll
    for (int j = 0; j < kCT; ++j) {
      acc[i][j] = floatx4{};
      if constexpr (kTerm) xa[i][j] = xb[i][j] = floatx4{};
    }
  // The MFMAs of one step; `between(n)` runs after group n of them.
  auto multiply = [&](const Frags& f, auto between) {
    if constexpr (kFold == kElScaled || kFold == kTermFold || kFold == kHiFold) {
      half8 bs[kCT];
#pragma unroll
      for (int j = 0; j < kCT; ++j) bs[j] = kFold == kElScaled ? f.bh[j] * s8 : f.bh[j];
      static_for<kCT>([&](auto J) {
        constexpr int j = decltype(J)::value;
#pragma unroll
        for (int i = 0; i < kRT; ++i) acc[i][j] = mfma16(f.ah[i], bs[j], acc[i][j]);
        between(std::integral_constant<int, j>{});
      });
      if constexpr (kFold != kHiFold) {
        static_for<kCT>([&](auto J) {
          constexpr int j = decltype(J)::value;
#pragma unroll
          for (int i = 0; i < kRT; ++i) {
            floatx4& x = kTerm ? xa[kTerm ? i : 0][kTerm ? j : 0] : acc[i][j];
            x = mfma16(f.al[i], f.bh[j], x);
          }
          between(std::integral_constant<int, kCT + j>{});
        });
        static_for<kCT>([&](auto J) {
          constexpr int j = decltype(J)::value;
#pragma unroll
          for (int i = 0; i < kRT; ++i) {
            floatx4& x = kTerm ? xb[kTerm ? i : 0][kTerm ? j : 0] : acc[i][j];
            x = mfma16(f.ah[i], f.bl[j], x);
          }
          between(std::integral_constant<int, 2 * kCT + j>{});
        });
      }
    } else {
      const floatx4 zero{};
      static_for<kCT>([&](auto J) {
        constexpr int j = decltype(J)::value;
        floatx4 t1[kRT], t2[kRT];
        half8 bs{};
        if constexpr (kFold == kCrScaled) bs = f.bh[j] * s8;
#pragma unroll
        for (int i = 0; i < kRT; ++i) {
          if constexpr (kFold == kElUnscaled) acc[i][j] = mfma16(f.ah[i], f.bh[j], acc[i][j]);
          if constexpr (kFold == kCrUnscaled) t2[i] = mfma16(f.ah[i], f.bh[j], zero);
        }
#pragma unroll
        for (int i = 0; i < kRT; ++i) t1[i] = mfma16(f.al[i], f.bh[j], zero);
        between(std::integral_constant<int, 3 * j>{});
#pragma unroll
        for (int i = 0; i < kRT; ++i) {
          if constexpr (kFold == kElUnscaled) t2[i] = mfma16(f.ah[i], f.bl[j], zero);
          else t1[i] = mfma16(f.ah[i], f.bl[j], t1[i]);
        }
        between(std::integral_constant<int, 3 * j + 1>{});
        if constexpr (kFold == kCrScaled) {
#pragma unroll
          for (int i = 0; i < kRT; ++i) t1[i] = mfma16(f.ah[i], bs, t1[i]);
        }
        between(std::integral_constant<int, 3 * j + 2>{});
#pragma unroll
        for (int i = 0; i < kRT; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (kFold == kElUnscaled) {
              acc[i][j][e] = __builtin_fmaf(t1[i][e], g.inv_s, acc[i][j][e]);
              acc[i][j][e] = __builtin_fmaf(t2[i][e], g.inv_s, acc[i][j][e]);
            } else if constexpr (kFold == kCrScaled) {
              acc[i][j][e] += t1[i][e];
            } else {
              acc[i][j][e] += __builtin_fmaf(t1[i][e], g.inv_s, t2[i][e]);
            }
          }
      });
    }
  };
  constexpr int kGroups = kFold == kHiFold ? kCT : 3 * kCT;

  // Stages 0 .. kStages-1 are in flight before the loop; step t waits for
  // stage t+1, reads its fragments while the MFMAs of stage t run, and refills
  // the slot of stage t (every wave has read it before this step's barrier).
  // The copies go between groups of MFMAs.
#pragma unroll
  for (int t = 0; t < S::kStages; ++t)
#pragma unroll
    for (int i = 0; i < S::kDma; ++i) copy_one(t, t, i);
  wait_vmcnt<(S::kStages - 1) * S::kDma>();
  lds_barrier();
  Frags f[2];
  read(f[0], 0);
  int slot = 0;  // of stage t
  auto step = [&](int t, const Frags& cur, Frags& next) {
    SCHED_FENCE();
    wait_vmcnt<(S::kStages - 2) * S::kDma>();
    lds_barrier();
    const int old = slot;
    slot = slot + 1 == S::kStages ? 0 : slot + 1;
    read(next, slot);
    SCHED_FENCE();
    multiply(cur, [&](auto G) {
      constexpr int n = decltype(G)::value;
      constexpr int d0 = n * S::kDma / kGroups, d1 = (n + 1) * S::kDma / kGroups;
      if constexpr (d1 > d0) {
        SCHED_FENCE();
#pragma unroll
        for (int i = d0; i < d1; ++i) copy_one(t + S::kStages, old, i);
        SCHED_FENCE();
      }
    });
  };
  for (int t = 0; t < ksteps; t += 2) {
    step(t, f[0], f[1]);
    step(t + 1, f[1], f[0]);
  }
  // No LDS DMA may still be writing when the workgroup retires.
  wait_vmcnt<0>();

  const int col0 = tn * S::kBN + wn * S::kWCols + (lane & 15);
  const int row0 = tm * S::kBM + wm * S::kWRows + (lane >> 4) * 4;
  const bool full = (tm + 1) * S::kBM <= g.M && (tn + 1) * S::kBN <= g.N;
  auto value = [&](int i, int j, int r) {
    if constexpr (kTerm)
      return __builtin_fmaf(xb[kTerm ? i : 0][kTerm ? j : 0][r], g.inv_s,
                            __builtin_fmaf(xa[kTerm ? i : 0][kTerm ? j : 0][r], g.inv_s,
                                           acc[i][j][r]));
    else if constexpr (kFold == kElScaled || kFold == kCrScaled)
      return acc[i][j][r] * g.inv_s;
    else
      return acc[i][j][r];
  };
  if constexpr (kFold != kHiFold) {
    if (g.report && blockIdx.x == 0 && threadIdx.x == 0) *g.report = range_report_bits(g.range);
    if (g.row_max) {
      int p[kRT][4], q[kCT];
#pragma unroll
      for (int i = 0; i < kRT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = row0 + 16 * i + r;
          p[i][r] = row < g.M ? prescale_shift(g.row_max[row], g.exp_a) : 0;
        }
#pragma unroll
      for (int j = 0; j < kCT; ++j) {
        const int col = col0 + 16 * j;
        q[j] = col < g.N ? prescale_shift(g.col_max[col], g.exp_b) : 0;
      }
      store_tile16<kRT, kCT>(g.C, g.ldc, g.M, g.N, row0, col0, full, [&](int i, int j, int r) {
        return __builtin_ldexpf(value(i, j, r), -(p[i][r] + q[j]));
      });
      return;
    }
  }
  store_tile16<kRT, kCT>(g.C, g.ldc, g.M, g.N, row0, col0, full, value);
}

template <int V, int kBM, int kBN, int kWM, int kWN, int kStages>
__global__ __launch_bounds__(64 * kWM * kWN, 1) void gemm_small_kernel(SmallArgs g,
                                                                       int unscaled_only) {
  using S = SmallShape<kBM, kBN, kWM, kWN, kStages, V == kHiOnly>;
  extern __shared__ __align__(16) uint16_t lds[];
  if constexpr (V == kTermwise) {
    small_tile<S, kTermFold>(g, lds);
  } else if constexpr (V == kHiOnly) {
    small_tile<S, kHiFold>(g, lds);
  } else {
    // The scaled body needs a finite s B_hi (gemm.hip): s <= 2^15 (host) and a
    // clear range flag.
    if (unscaled_only || g.range[0] == g.range[1])
      small_tile<S, V == kElementwise ? kElUnscaled : kCrUnscaled>(g, lds);
    else
      small_tile<S, V == kElementwise ? kElScaled : kCrScaled>(g, lds);
  }
}

template <int V, int kBM, int kBN, int kWM, int kWN, int kStages>
hipError_t launch_small(const Planes& p, int64_t M, int64_t N, float* C, int64_t ldc, float s,
                        hipStream_t stream, const RangeOpts& opt, uint32_t* report) {
  using S = SmallShape<kBM, kBN, kWM, kWN, kStages, V == kHiOnly>;
  static std::atomic<bool> done[kMaxDevices];
  const hipError_t attr =
      set_lds(&gemm_small_kernel<V, kBM, kBN, kWM, kWN, kStages>, S::kLdsBytes, done);
  if (attr != hipSuccess) return attr;
  SmallArgs g{p.a_hi, p.a_lo, p.b_hi, p.b_lo, p.range, static_cast<int>(p.Kp),
              static_cast<int>((M + kBM - 1) / kBM), static_cast<int>((N + kBN - 1) / kBN),
              C, ldc, static_cast<int>(M), static_cast<int>(N), s, 1.0f / s,
              opt.prescale ? p.row_max : nullptr, opt.prescale ? p.col_max : nullptr,
              opt.exp_a, opt.exp_b, report};
  hipLaunchKernelGGL((gemm_small_kernel<V, kBM, kBN, kWM, kWN, kStages>),
                     dim3(g.tiles_m * g.tiles_n), dim3(S::kThreads), S::kLdsBytes, stream, g,
                     scaled_kernel_ok(s) ? 0 : 1);
  return hipGetLastError();
}

template <int V>
hipError_t launch_config(int tile, const Planes& p, int64_t M, int64_t N, float* C, int64_t ldc,
                         float s, hipStream_t stream, const RangeOpts& opt, uint32_t* report) {
  switch (tile) {
    case 32: return launch_small<V, 32, 32, 2, 2, 8>(p, M, N, C, ldc, s, stream, opt, report);
    case 64:
      if constexpr (V == kHiOnly)
        return launch_small<V, 64, 64, 2, 2, 8>(p, M, N, C, ldc, s, stream, opt, report);
      else
        return launch_small<V, 64, 64, 4, 2, 4>(p, M, N, C, ldc, s, stream, opt, report);
    case 128:
      return launch_small<V, 128, 128, 2, 4, 4>(p, M, N, C, ldc, s, stream, opt, report);
    default: return hipErrorInvalidValue;
  }
}

// Microseconds per 32-wide k-step of a grid of `tiles` workgroups, one per
// compute unit at a time: each round of 256 costs `base` plus `fill` times the
// share of the chip it occupies (fuller rounds run slower: they share the
// power limit and the caches).
double grid_cost(int64_t tiles, double base, double fill) {
  const int64_t rounds = tiles / 256, rest = tiles % 256;
  return rounds * (base + fill) + (rest ? base + fill * rest / 256.0 : 0.0);
}

}  // namespace

// The rule: the tile whose grid costs least.  The constants (indexed by Variant)
// were fitted to the kernels' times on 75 grids from 256 x 256 to 16384 x 512
// at K = 512 to 2048; on those grids the pick is the fastest tile or within
// 10 % of it.  Where the lines lie for the elementwise order, 64 k-steps: 32
// up to 512 tiles of 32 (512 x 1024: 15.9 against 19.4 us on 64-wide tiles;
// 512 x 1280: 23.7 against 19.4), then 64 up to 512 tiles of 64 (1024 x 2048:
// 34.5 against 43.0 on 128; 768 x 3072: 46.7 against 44.3), then 128 while its
// rounds are fuller than those of the wide tiles (2048 x 4096: 96.8 against
// 122.9; 2560 x 4096: 136 against 123).
int small_gemm_tile(int64_t M, int64_t N, int variant) {
  auto tiles = [&](int64_t bm, int64_t bn) {
    return ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  };
  struct Cost {
    double base, fill;
  };
  static constexpr Cost k32[4] = {{0.105, 0.005}, {0.095, 0.005}, {0.055, 0.005}, {0.11, 0.01}};
  static constexpr Cost k64[4] = {{0.215, 0.02}, {0.20, 0.03}, {0.115, 0.01}, {0.23, 0.02}};
  static constexpr Cost k128[4] = {{0.54, 0.18}, {0.52, 0.19}, {0.20, 0.06}, {0.56, 0.20}};
  static constexpr Cost kBig[4] = {{1.57, 0.60}, {0.83, 0.38}, {0.66, 0.29}, {0.95, 0.40}};
  const bool wide = variant == kElementwise || variant == kHiOnly;
  const double c32 = grid_cost(tiles(32, 32), k32[variant].base, k32[variant].fill);
  const double c64 = grid_cost(tiles(64, 64), k64[variant].base, k64[variant].fill);
  const double c128 = grid_cost(tiles(128, 128), k128[variant].base, k128[variant].fill);
  const double big = grid_cost(tiles(256, wide ? 256 : 128), kBig[variant].base, kBig[variant].fill);
  const double best = std::min(std::min(c32, c64), std::min(c128, big));
  return best == big ? 0 : best == c128 ? 128 : best == c64 ? 64 : 32;
}

hipError_t launch_gemm_small(int tile, const Planes& p, int64_t M, int64_t N, float* C,
                             int64_t ldc, float scale, int variant, hipStream_t stream,
                             const RangeOpts& opt, uint32_t* report) {
  switch (variant) {
    case kElementwise:
      return launch_config<kElementwise>(tile, p, M, N, C, ldc, scale, stream, opt, report);
    case kTermwise:
      return launch_config<kTermwise>(tile, p, M, N, C, ldc, scale, stream, opt, report);
    case kCrossFirst:
      return launch_config<kCrossFirst>(tile, p, M, N, C, ldc, scale, stream, opt, report);
    case kHiOnly:
      return launch_config<kHiOnly>(tile, p, M, N, C, ldc, scale, stream, opt, report);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sgc
