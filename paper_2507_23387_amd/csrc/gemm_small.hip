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
// over more compute units but moves more LDS bytes per MFMA.  A 64 x 64 step is
// 192 cycles of MFMAs per SIMD, 256 cycles of LDS reads and 128 of the copies'
// LDS writes at 128 B per clock, and a barrier, and takes about 500 cycles (0.23
// us; without the copies 25 of 31 us at 1024 x 1024 x 4096 termwise, without the
// reads 28, without both 19).  A 32 x 32 step takes 0.1 us, most of it the
// barrier and an LDS read's latency.  So the tile is the smallest that still
// leaves few workgroups per compute unit.  GEMM alone, wide kernel against this
// one: elementwise 256^3 25.8 and 4.0 us, 300 x 200 x 1024 61 and 6.2, 1024^3
// 60 and 11.2, 48 x 4096 x 4096 196 and 17.4, 2048 x 2048 x 2816 141 and 59;
// termwise 34.4 and 10.3 at 1024^3; the FP16 baseline 70 and 27 at 2048 x 2048
// x 2816.
#include <algorithm>
#include <atomic>
#include <cmath>

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
  static_assert(kBM % 32 == 0 && kBN % 32 == 0, "tiles are whole 32-row pieces");
  static_assert(kWRows % 16 == 0 && kWCols % 16 == 0, "whole MFMA tiles per wave");
  static_assert(kUnits % kWaves == 0, "every wave issues the same number of copies");
  static_assert(kStages >= 2, "the ring holds the stage multiplied, then refilled, and the one read");
  static_assert(kLdsBytes <= kMaxLdsBytes, "LDS of every kernel stays within 128 KiB");
};

struct SmallArgs {
  const uint16_t* a_hi;
  const uint16_t* a_lo;
  const uint16_t* b_hi;
  const uint16_t* b_lo;
  const uint32_t* range;
  int Mp, Np, Kp, tiles_m, tiles_n;
  bool by_xcd;
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
  if (S::kBM < 256 || !tile_of_block(blockIdx.x, g.tiles_m, g.tiles_n, tm, tn))
    tile_of<4>(g.by_xcd ? xcd_order(blockIdx.x, g.tiles_m * g.tiles_n) : blockIdx.x, g.tiles_m,
               g.tiles_n, tm, tn);
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
    // Tiles that are not whole panels can reach past the plane's padded rows
    // (M and N rounded up to 256): those rows' results are never stored, and
    // their copies repeat the plane's last 32 rows.
    const int row = min((is_a ? tm * S::kBM : tn * S::kBN) + 32 * r, (is_a ? g.Mp : g.Np) - 32);
    const uint16_t* plane = is_a ? (p ? g.a_lo : g.a_hi) : (p ? g.b_lo : g.b_hi);
    src[i] = reinterpret_cast<const char*>(plane) + (row / kPanel) * panel_bytes +
             sl * (kTileHalves * 2) + (row % kPanel) * (kSlice * 2);
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
  constexpr bool kScaled = kFold == kElScaled || kFold == kCrScaled;
  struct Frags {
    half8 ah[kRT], al[kRT], bh[kCT], bl[kCT];
    half8 bs[kScaled ? kCT : 1];  // s B_hi, exact (gemm.hip)
  };
  // Read r of a step's fragments: B_hi, A_hi, A_lo, B_lo, the order of first use.
  auto read_one = [&](Frags& f, int slot, auto Rc) {
    constexpr int r = decltype(Rc)::value;
    if constexpr (r < kCT) f.bh[r] = rd_b(slot, 0, r);
    else if constexpr (r < kCT + kRT) f.ah[r - kCT] = rd_a(slot, 0, r - kCT);
    else if constexpr (r < kCT + 2 * kRT) f.al[r - kCT - kRT] = rd_a(slot, 1, r - kCT - kRT);
    else f.bl[r - kCT - 2 * kRT] = rd_b(slot, 1, r - kCT - 2 * kRT);
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
  // The MFMAs of one step, in the order of gemm.hip's kernels per accumulator;
  // `after(m)` runs after the m-th of them.
  constexpr int kTile = kRT * kCT;
  constexpr int kMfmas = kFold == kHiFold ? kTile : 3 * kTile;
  auto multiply = [&](const Frags& f, auto after) {
    if constexpr (kFold == kElScaled || kFold == kTermFold || kFold == kHiFold) {
      static_for<kMfmas>([&](auto Mc) {
        constexpr int m = decltype(Mc)::value, g = m / kTile, j = m % kTile / kRT, i = m % kRT;
        if constexpr (g == 0) {
          acc[i][j] = mfma16(f.ah[i], kFold == kElScaled ? f.bs[kScaled ? j : 0] : f.bh[j], acc[i][j]);
        } else if constexpr (g == 1) {
          floatx4& x = kTerm ? xa[kTerm ? i : 0][kTerm ? j : 0] : acc[i][j];
          x = mfma16(f.al[i], f.bh[j], x);
        } else {
          floatx4& x = kTerm ? xb[kTerm ? i : 0][kTerm ? j : 0] : acc[i][j];
          x = mfma16(f.ah[i], f.bl[j], x);
        }
        after(Mc);
      });
    } else {
      const floatx4 zero{};
      static_for<kCT>([&](auto J) {
        constexpr int j = decltype(J)::value;
        floatx4 t1[kRT], t2[kRT];
        static_for<3 * kRT>([&](auto Mc) {
          constexpr int m = decltype(Mc)::value, g = m / kRT, i = m % kRT;
          if constexpr (kFold == kElUnscaled) {
            if constexpr (g == 0) acc[i][j] = mfma16(f.ah[i], f.bh[j], acc[i][j]);
            else if constexpr (g == 1) t1[i] = mfma16(f.al[i], f.bh[j], zero);
            else t2[i] = mfma16(f.ah[i], f.bl[j], zero);
          } else if constexpr (kFold == kCrScaled) {
            if constexpr (g == 0) t1[i] = mfma16(f.al[i], f.bh[j], zero);
            else if constexpr (g == 1) t1[i] = mfma16(f.ah[i], f.bl[j], t1[i]);
            else t1[i] = mfma16(f.ah[i], f.bs[kScaled ? j : 0], t1[i]);
          } else {
            if constexpr (g == 0) t2[i] = mfma16(f.ah[i], f.bh[j], zero);
            else if constexpr (g == 1) t1[i] = mfma16(f.al[i], f.bh[j], zero);
            else t1[i] = mfma16(f.ah[i], f.bl[j], t1[i]);
          }
          after(std::integral_constant<int, 3 * kRT * j + m>{});
        });
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

  // Stages 0 .. kStages-1 are in flight before the loop; step t waits for
  // stage t+1, reads its fragments while the MFMAs of stage t run, and refills
  // the slot of stage t (every wave has read it before this step's barrier).
#pragma unroll
  for (int t = 0; t < S::kStages; ++t)
#pragma unroll
    for (int i = 0; i < S::kDma; ++i) copy_one(t, t, i);
  wait_vmcnt<(S::kStages - 1) * S::kDma>();
  lds_barrier();
  // A burst of LDS reads or of copies holds the wave's issue for as long as the
  // LDS or the copy engine takes to serve all waves', so the reads of the next
  // step go one after each MFMA (more where a step has fewer MFMAs than reads).
  // The copies go after the reads, or, where a wave has 8 or more accumulators,
  // evenly over the step (2048 x 2048 x 2816 on 128-wide tiles 59 us so, 62
  // after the reads; 1024 x 1024 x 4096 on 64-wide tiles 36 and 32).
  constexpr int kReads = (kFold == kHiFold ? 1 : 2) * (kRT + kCT);
  constexpr int kReadsPer = (kReads + kMfmas - 1) / kMfmas;
  Frags f[2];
  static_for<kReads>([&](auto Rc) { read_one(f[0], 0, Rc); });
  if constexpr (kScaled) {
#pragma unroll
    for (int j = 0; j < kCT; ++j) f[0].bs[j] = f[0].bh[j] * s8;
  }
  int slot = 0;  // of stage t
  auto step = [&](int t, const Frags& cur, Frags& next) {
    SCHED_FENCE();
    wait_vmcnt<(S::kStages - 2) * S::kDma>();
    lds_barrier();
    const int refill = slot;
    slot = slot + 1 == S::kStages ? 0 : slot + 1;
    SCHED_FENCE();
    multiply(cur, [&](auto Mc) {
      constexpr int m = decltype(Mc)::value;
      SCHED_FENCE();
      static_for<kReadsPer>([&](auto Rc) {
        constexpr int r = m * kReadsPer + decltype(Rc)::value;
        if constexpr (r < kReads) read_one(next, slot, std::integral_constant<int, r>{});
      });
      constexpr int kReadSlots = (kReads + kReadsPer - 1) / kReadsPer;
      constexpr int kFirst = kTile >= 8 ? 0 : kReadSlots < kMfmas ? kReadSlots : kMfmas - 1;
      // A ring of two waits for this step's copies at the next barrier: they go
      // into its first half.
      constexpr int kSlots = S::kStages == 2 ? kMfmas / 2 : kMfmas - kFirst, n = m - kFirst;
      constexpr int d0 = n < 0 || n >= kSlots ? 0 : n * S::kDma / kSlots;
      constexpr int d1 = n < 0 || n >= kSlots ? 0 : (n + 1) * S::kDma / kSlots;
#pragma unroll
      for (int i = d0; i < d1; ++i) copy_one(t + S::kStages, refill, i);
      // s B_hi of the next step, of whose reads B_hi came first, after the last
      // MFMAs of this one.
      if constexpr (kScaled && m >= kMfmas - kCT) {
        constexpr int j = m - (kMfmas - kCT);
        next.bs[j] = next.bh[j] * s8;
      }
      SCHED_FENCE();
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

// The unscaled body alone, on 256 x 128 tiles: the fallback of the 256-wide
// scaled kernels (gemm.hip).  Unless the host routed the call here (unscaled_only:
// s is not a finite FP16 value) it returns at once where the range flag is
// clear.  Two waves per SIMD, so that one's folds (32 vector operations per 12
// MFMAs) run beside the other's MFMAs: 4096 x 4096 x 16384 elementwise 1338 us,
// cross-first 1340, against 1395 and 1429 for one wave per SIMD with the folds
// placed between the MFMAs by hand (8192^3: 2742 against 2780, 2727 against 2821).
using UnscaledShape = SmallShape<256, 128, 4, 2, 2, false>;
template <int V>
__global__ __launch_bounds__(512, 1) void gemm_unscaled_kernel(SmallArgs g, int unscaled_only) {
  extern __shared__ __align__(16) uint16_t lds[];
  if (!unscaled_only && g.range[0] != g.range[1]) return;
  small_tile<UnscaledShape, V == kElementwise ? kElUnscaled : kCrUnscaled>(g, lds);
}

template <class S>
SmallArgs small_args(const Planes& p, int64_t M, int64_t N, float* C, int64_t ldc, float s,
                     const RangeOpts& opt, uint32_t* report) {
  const int tiles_m = static_cast<int>((M + S::kBM - 1) / S::kBM);
  const int tiles_n = static_cast<int>((N + S::kBN - 1) / S::kBN);
  // In a grid that is no multiple of 8 the tiles of one column lie on different
  // XCDs, each of which reads B's panel for itself.  Consecutive tiles for each
  // XCD pay where a few rows of tiles read a B that its L2s do not hold: termwise
  // 151 x 7265 x 4096 on 64-wide tiles 66 us without, 47 with; 298 x 13008 x 3273
  // 121 and 98; of 273 such problems 9 % faster on average, the slowest by 6 %.
  // One row of tiles shares no B (28 x 832 x 54592 144 without, 200 with), and
  // many rows, few columns lose too (37086 x 68 x 1152 40 and 79).
  const bool by_xcd = S::kBM < 256 && tiles_m * tiles_n % 8 != 0 && tiles_m >= 3 &&
                      tiles_n >= 2 * tiles_m && p.Np * p.Kp * 4 >= (16 << 20);
  return SmallArgs{p.a_hi, p.a_lo, p.b_hi, p.b_lo, p.range, static_cast<int>(p.Mp),
                   static_cast<int>(p.Np), static_cast<int>(p.Kp), tiles_m, tiles_n, by_xcd, C,
                   ldc, static_cast<int>(M),
                   static_cast<int>(N), s, 1.0f / s, opt.prescale ? p.row_max : nullptr,
                   opt.prescale ? p.col_max : nullptr, opt.exp_a, opt.exp_b, report};
}

template <int V>
hipError_t launch_unscaled(const Planes& p, int64_t M, int64_t N, float* C, int64_t ldc, float s,
                           bool only, hipStream_t stream) {
  using S = UnscaledShape;
  static std::atomic<bool> done[kMaxDevices];
  const hipError_t attr = set_lds(&gemm_unscaled_kernel<V>, S::kLdsBytes, done);
  if (attr != hipSuccess) return attr;
  const SmallArgs g = small_args<S>(p, M, N, C, ldc, s, RangeOpts{}, nullptr);
  hipLaunchKernelGGL(gemm_unscaled_kernel<V>, dim3(g.tiles_m * g.tiles_n), dim3(S::kThreads),
                     S::kLdsBytes, stream, g, only ? 1 : 0);
  return hipGetLastError();
}

template <int V, int kBM, int kBN, int kWM, int kWN, int kStages>
hipError_t launch_small(const Planes& p, int64_t M, int64_t N, float* C, int64_t ldc, float s,
                        hipStream_t stream, const RangeOpts& opt, uint32_t* report) {
  using S = SmallShape<kBM, kBN, kWM, kWN, kStages, V == kHiOnly>;
  static_assert(S::kThreads == small_tile_threads(kBM, V), "the rule counts these threads");
  static std::atomic<bool> done[kMaxDevices];
  const hipError_t attr =
      set_lds(&gemm_small_kernel<V, kBM, kBN, kWM, kWN, kStages>, S::kLdsBytes, done);
  if (attr != hipSuccess) return attr;
  const SmallArgs g = small_args<S>(p, M, N, C, ldc, s, opt, report);
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
      // Four waves of 32 x 32 read fewer LDS bytes per MFMA than eight of 16 x
      // 32 (1024 x 1024 x 4096: elementwise 32 against 37 us); the cross-first
      // folds keep eight, whose vector adds overlap the other wave's MFMAs (39
      // against 41).
      if constexpr (V == kCrossFirst)
        return launch_small<V, 64, 64, 4, 2, 4>(p, M, N, C, ldc, s, stream, opt, report);
      else
        return launch_small<V, 64, 64, 2, 2, 4>(p, M, N, C, ldc, s, stream, opt, report);
    case 192:
      // Orders of one accumulator set: eight waves of 48 x 96 fit both steps'
      // fragments in VGPRs (four of 96 x 96 move the accumulators of the folds
      // in and out of AGPRs: cross-first 3072 x 3072 x 2048 129 us against 98).
      if constexpr (V == kElementwise || V == kCrossFirst)
        return launch_small<V, 192, 192, 4, 2, 2>(p, M, N, C, ldc, s, stream, opt, report);
      else
        return hipErrorInvalidValue;
    case 128:
      return launch_small<V, 128, 128, 2, 4, 4>(p, M, N, C, ldc, s, stream, opt, report);
    default: return hipErrorInvalidValue;
  }
}

// Time of a grid, in microseconds: `launch`, plus `start` (a tile's prologue and
// its stores) per round of workgroups that run together, plus for each 32-wide
// k-step `round` per round and `tile` per workgroup of each compute unit
// (fuller grids share caches and the power limit).
struct GridCost {
  double launch, start, round, tile;
};
double grid_time(const GridCost& c, int64_t tiles, int64_t together, int64_t ksteps) {
  const int64_t rounds = (tiles + together - 1) / together;
  return c.launch + rounds * (c.start + ksteps * c.round) + ksteps * c.tile * tiles / 256;
}

}  // namespace

// The rule: the tile whose grid takes the least time, and the 256-wide kernels
// where they come within 5 % of it (baseline: 10 %).  The constants (indexed by
// Variant) are a least-squares fit to the kernels' times on 2335 problems per
// order, from 16 to 16384 rows and columns at K = 64 to 16384
// (profiles/tile_rule_grids.csv).  Over those the pick's GEMM is 0.3-0.9 % slower
// than the fastest tile's on average, and slower than the 256-wide kernels' by
// more than 5 % on 2 of the 9340.  Without `start` and the margin
// it was 1.6-3.4 %, and 231 problems ran up to 40 % slower than on the 256-wide
// kernels, most of them where those fill a round or two at small K (termwise 1024
// x 8192 x 512: 33-35 us on 128-wide tiles, 29-30).  What is left is mostly
// operand traffic, which the model leaves out (62 x 8118 x 4096 elementwise: 52
// us on 32-wide tiles, 30 on 64).  The fifth constants are those of the unscaled
// elementwise body, for s > 2^15: its folds make 64-wide tiles, of one wave per
// SIMD, half again as slow (762 x 5771 x 2048: 105 us on them, 80 on 256 x 128);
// with the others' constants 124 of 1666 problems ran more than 5 % slower than
// on the 256-wide kernel, now none.  A call whose range flag is set runs the same
// body on the tile picked for the scaled one.
// Two workgroups of 32 or 64-wide tiles share a compute unit (64 KiB of LDS
// each), so their rounds are of 512.  Where the lines lie for the elementwise
// order at K = 2048: 32 up to 512 tiles of 32 (512 x 1024: 15.9 us against 18.6
// on 64-wide tiles; 512 x 1280: 23.6 against 18.9), then 64 up to 512 tiles of 64
// (1024 x 2048: 33.8 against 37.6 on 128; 768 x 3072: 45 against 39), then 128
// while the wide tiles' rounds are emptier (2048 x 4096: 91 against 123).
// 192-wide tiles take the grids between 256 tiles of 128 and 256 of 256 (3072 x
// 3072: 90 us, 118 on 128 and 115 on wide ones; 5760 x 5760 x 4096: 652 against
// 712).
int small_gemm_tile(int64_t M, int64_t N, int64_t K, int variant, bool unscaled,
                    double split_us) {
  static constexpr GridCost k32[5] = {{2.0, 1.56, 0.083, 0.050},
                                      {2.2, 1.31, 0.067, 0.050},
                                      {3.1, 0.32, 0.053, 0.014},
                                      {2.3, 1.37, 0.100, 0.043},
                                      {2.1, 1.44, 0.124, 0.036}};
  static constexpr GridCost k64[5] = {{2.0, 2.70, 0.124, 0.141},
                                      {1.6, 2.79, 0.113, 0.137},
                                      {2.5, 1.22, 0.089, 0.049},
                                      {1.8, 2.45, 0.149, 0.149},
                                      {1.7, 2.37, 0.256, 0.154}};
  static constexpr GridCost k128[5] = {{2.2, 4.38, 0.356, 0.258},
                                       {1.7, 4.61, 0.327, 0.274},
                                       {2.2, 2.37, 0.156, 0.072},
                                       {2.2, 4.30, 0.394, 0.281},
                                       {1.8, 3.86, 0.459, 0.281}};
  static constexpr GridCost k192[5] = {{2.5, 7.53, 0.772, 0.479},
                                       {},
                                       {},
                                       {2.7, 7.55, 0.867, 0.503},
                                       {1.9, 7.05, 0.859, 0.575}};
  static constexpr GridCost kWide[5] = {{4.2, 13.14, 1.306, 0.618},
                                        {2.9, 9.05, 0.660, 0.397},
                                        {1.6, 11.56, 0.601, 0.199},
                                        {4.4, 6.95, 0.790, 0.435},
                                        {2.1, 6.92, 0.809, 0.496}};
  const int row = unscaled && variant == kElementwise ? 4 : variant;
  auto time = [&](const GridCost& c, int64_t bm, int64_t bn, int64_t together) {
    const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
    // A grid dimension holds less than 2^32 threads, which 32-wide tiles reach
    // at M = 2^29 (137 GB of planes at K <= 64); the 256-wide kernels have room
    // for every problem whose C fits a device.
    if (bm < 256 && tiles * small_tile_threads(static_cast<int>(bm), variant) > UINT32_MAX)
      return HUGE_VAL;
    return grid_time(c, tiles, together, round_up(K, kKPad) / kSmallStep);
  };
  const bool square = row == kElementwise || row == kHiOnly;
  // Machines differ by a few percent, and past one round the model is too kind to
  // the small tiles of the baseline.
  const double wide = time(kWide[row], 256, square ? 256 : 128, 256);
  double limit = (variant == kHiOnly ? 0.90 : 0.95) * wide;
  // Splitting A costs the 256-wide kernels 5 % (32768 x 256 x 1024 elementwise 76
  // us; a pass over A and 128-wide tiles 97; 8192 x 1024 x 1024 the other way, 74
  // and 64; termwise 16384 x 256 x 1024 42 and 47, 8192 x 256 x 4096 122 and 100).
  // On few workgroups the termwise kernel loses more (13632 x 1 x 16832: 614 us,
  // 535 on tiles).
  if (split_us > 0)
    limit = std::min(limit, (variant == kTermwise ? 1.10 : 1.05) * wide - split_us);
  // Planes of A that the 256 MiB last-level cache cannot hold come back from HBM,
  // at the rate they went (27840 x 5 x 8832 elementwise: 496 us on the 256-wide
  // kernel, 532 on 32-wide tiles).  Not termwise, whose 256 x 128 kernel splits a
  // long A slower than that (13056 x 2 x 17920: 609 us, 540 on tiles).
  const double read_us =
      variant == kElementwise && 4.0 * M * K > 256.0 * (1 << 20) ? 0.5 * split_us : 0.0;
  int tile = 0;
  auto consider = [&](int side, double us) {
    us = std::max(us, read_us);
    if (us < limit) limit = us, tile = side;
  };
  consider(32, time(k32[row], 32, 32, 512));
  consider(64, time(k64[row], 64, 64, 512));
  consider(128, time(k128[row], 128, 128, 256));
  if (variant == kElementwise || variant == kCrossFirst)
    consider(192, time(k192[row], 192, 192, 256));
  return tile;
}

hipError_t launch_gemm_unscaled(const Planes& p, int64_t M, int64_t N, float* C, int64_t ldc,
                                float scale, int variant, bool only, hipStream_t stream) {
  switch (variant) {
    case kElementwise:
      return launch_unscaled<kElementwise>(p, M, N, C, ldc, scale, only, stream);
    case kCrossFirst: return launch_unscaled<kCrossFirst>(p, M, N, C, ldc, scale, only, stream);
    default: return hipErrorInvalidValue;
  }
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
