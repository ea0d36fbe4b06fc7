// Symmetric-output split products of small orders, whose 256 x 256 tiles
// would leave the machine idle.  A work-group owns one square tile of 32, 64
// or 96 rows on or above the diagonal and its waves split the K range: every wave
// computes the whole tile over its own piece, with fragments loaded straight
// from the K-tiled planes into registers (a fragment is two contiguous
// 512-byte runs, and no two waves share one, so LDS would only add a copy and a
// barrier per step).  The waves' partial tiles meet in LDS, a 32-row strip at
// a time, where the epilogue finishes them: one launch per product, no partial
// accumulators in memory.  The pieces are those of the split-K plan of the
// 256 x 256 kernel and are summed in their order, so a product is the same bit
// for bit as there, but for two-segment products of n = 769 to 1280, whose plan
// has 16 or 17 pieces and a work-group at most 12 waves (error of a BF16X3
// derivative of those orders: 1.00 times that of the plan).  At n = 402 (32-row tiles, 4 waves) a layer takes 8.6 us
// against 25.8 us in the 256 x 256 kernel and its split-K strip kernel, at
// n = 1026 17.7 against 35.6 us, at n = 2046 (96-row tiles, 7 waves) 42 against
// 58.6 us.  At 402 and 1026 that is a decision head of 2 us, a K loop of 0.3 to
// 4 us, an epilogue of 2 to 5 us and the gap between launches; at 2046 the K loop
// takes 26 us: 389 MB of fragments come out of L2 at 15 TB/s, so a larger tile
// than the registers hold (9 of 32 x 32 and two K steps, two waves per SIMD)
// would be needed to go on.
#pragma once

#include <type_traits>

#include "sp2_common.hpp"
#include "sp2_gemm.hpp"

namespace sp2 {

// Operand kind of the FP32 products (k_wave_f32).
constexpr int kF32 = 3;

// Products of a split kind: main term first, the small cross terms after it.
template <int KIND>
struct KindTraits {
  static constexpr int planes = KIND == kBF16X1 ? 1 : 2;
  static constexpr int products = KIND == kBF16X1 ? 1 : 3;
};

// Tile schedule of a launch: nt tile rows of 32 MB rows; nw K pieces, one per
// wave (at least WaveShape::kMinWaves waves, those past nw without a piece);
// operand rows and columns at or past lim (a multiple of 64) are zero.
struct WaveGrid {
  int nt, ntiles, band;
  int nw;
  int lim;
};

struct WaveArgs {
  const uint16_t* a[2][2];   // [segment][plane]
  const uint16_t* b[2][2];
  Epi epi;
  Decide dec;
  WaveGrid g;
};

// plane_off in 32 bits (np < 65536).
__device__ __forceinline__ uint32_t plane_off32(int i, int k, int np) {
  const uint32_t blk = uint32_t(i >> 8) * uint32_t(np >> 4) + uint32_t(k >> 4);
  return blk * 4096u + uint32_t(((k >> 3) & 1) * 2048 + (i & 255) * 8 + (k & 7));
}

template <int MB>
struct WaveShape {
  static constexpr int T = 32 * MB;
  // LDS: the image [T][LD] (odd stride: rows and columns conflict free) and
  // one 32-row strip of every wave's partial tile [nw][T][LP]
  static constexpr int LD = T + 1, LP = 36;
  static constexpr int kMinWaves = MB < 3 ? 4 : 6, kMaxWaves = MB < 3 ? 12 : 8;
  static constexpr int kImg = (T * LD + 3) & ~3, kLds = kImg + kMaxWaves * T * LP;
  // four-row groups of a strip per thread, of at least `waves` waves
  static constexpr int groups(int waves) { return (8 * T + waves * kWave - 1) / (waves * kWave); }
  static constexpr int Q = groups(kMinWaves);
};
constexpr int kWaveMaxWaves = 12;

// Decision of a layer by every wave for itself, every load issued at once:
// the stop flag, the control words and the trace partials arrive together
// (each is a round trip to memory that another XCD wrote), and no barrier is
// needed.  A wave that reads the flag as work-group 0 of this very launch sets
// it leaves as the others do: they find the same stop in the same sums.
__device__ __forceinline__ LayerCoef decide_layer_wave(const Decide& d) {
  if (d.mode == 2 || d.mode == 3) return hist_coef(d.hist, d.layer, d.mode == 2);
  if (d.mode != 1) return LayerCoef{1, 1.0f, 0.0f, 0.0f};
  const int n = d.layer;
  const int stopped = __atomic_load_n(&d.ctrl->stopped, __ATOMIC_RELAXED);
  const int acc_len = d.ctrl->acc_len, stall_from = d.ctrl->stall_from;
  const LayerCoef hc = hist_coef(d.hist, n, true);
  const double ep = err_before(d.hist->err, n);
  double t1 = 0.0, t2 = 0.0;
#pragma clang loop unroll_count(4)
  for (int i = threadIdx.x & (kWave - 1); i < d.nparts_in; i += kWave) {
    t1 += d.parts_in[2 * i];
    t2 += d.parts_in[2 * i + 1];
  }
  t1 = wave_total(t1);
  t2 = wave_total(t2);
  if (__builtin_amdgcn_readfirstlane(stopped)) {
    post_stopped(d);
    return LayerCoef{0, 0.0f, 0.0f, 0.0f};
  }
  return decide_from_sums(d, t1, t2, acc_len, stall_from, ep, hc);
}

template <int KIND>
__device__ __forceinline__ void mfma_32x32x16(f32x16& acc, u32x4 a, u32x4 b) {
  if constexpr (KIND == kFP16X3)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                 __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
  else
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

template <int KIND, int MB>
struct WaveFrag {
  u32x4 a[KindTraits<KIND>::planes][MB];
  u32x4 b[KindTraits<KIND>::planes][MB];
};

template <int KIND, int MB>
__device__ __forceinline__ void wave_products(const WaveFrag<KIND, MB>& f, f32x16 (&acc)[MB][MB]) {
  constexpr int pa[3] = {0, 0, 1}, pb[3] = {0, 1, 0};   // hi hi, hi lo, lo hi
#pragma clang loop unroll(full)
  for (int k = 0; k < KindTraits<KIND>::products; ++k)
#pragma clang loop unroll(full)
    for (int mi = 0; mi < MB; ++mi)
#pragma clang loop unroll(full)
      for (int ni = 0; ni < MB; ++ni)
        mfma_32x32x16<KIND>(acc[mi][ni], f.a[pa[k]][mi], f.b[pb[k]][ni]);
}

// C of this thread: four rows of one column per group, strip mi of the tile.
template <int MB, int Q>
__device__ __forceinline__ void wave_load_c(f32x4 (&cv)[Q], const Epi& p, int R0, int C0, int mi) {
  constexpr int T = WaveShape<MB>::T;
  const int np = p.np, nt = blockDim.x;
#pragma clang loop unroll(full)
  for (int i = 0; i < Q; ++i) {
    const int q = threadIdx.x + nt * i, col = C0 + q % T, row = R0 + 32 * mi + q / T * 4;
    const float* c = p.c + int64_t(row) * np + col;
    const bool in = p.c && q < 8 * T && (MB < 3 || (row < np && col < np));
#pragma clang loop unroll(full)
    for (int e = 0; e < 4; ++e) cv[i][e] = in ? c[int64_t(e) * np] : 0.0f;
  }
}

// What follows from the finished image of a tile (element (row, column) at
// column * CS + row * RS): the mirrored FP32 result, the planes, and the tile's
// trace pair.
template <int KIND, int T, int CS, int RS>
__device__ __forceinline__ void tile_finish(const Epi& p, int R0, int C0, int w, int lane,
                                            const float* img, double* red, int tile, double t1,
                                            double t2) {
  const int np = p.np, nv = p.n_valid, NT = blockDim.x, t = threadIdx.x;
  const bool diag = R0 == C0;
  if (p.out && p.mirror_out) {
    // row C0 + c, columns R0 + r .. r + 3
#pragma clang loop unroll(disable)
    for (int q = t; q < T * T / 4; q += NT) {
      const int r = (q % (T / 4)) * 4, c = q / (T / 4);
      const int row = C0 + c, col = R0 + r;
      float* o = p.out + int64_t(row) * p.ld_out + col;
      const float* s = img + c * CS + r * RS;
      if (row >= nv || col >= nv) continue;
      if (!diag && p.vec_ok && col + 3 < nv) {
        *reinterpret_cast<f32x4*>(o) = f32x4{s[0], s[RS], s[2 * RS], s[3 * RS]};
      } else {
#pragma clang loop unroll(disable)
        for (int e = 0; e < 4; ++e)
          if (col + e < nv && (!diag || r + e < c)) o[e] = s[e * RS];
      }
    }
  }
  // Planes: a thread per row and 8-column chunk (512-byte runs), then, off
  // the diagonal, the same of the mirror image.
  if constexpr (KIND != kF32) if (p.split_out) {
    constexpr int B = T * T / 8;
#pragma clang loop unroll_count(2)
    for (int q0 = t; q0 < (diag ? B : 2 * B); q0 += NT) {
      const bool mir = q0 >= B;
      const int q = mir ? q0 - B : q0;
      const int i = q % T, k = (q / T) * 8;
      const float* s = mir ? img + i * CS + k * RS : img + k * CS + i * RS;
      const int st = mir ? RS : CS;
      float v[8];
      if (CS == 1 && !mir) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(s), y = *reinterpret_cast<const f32x4*>(s + 4);
#pragma clang loop unroll(full)
        for (int e = 0; e < 4; ++e) {
          v[e] = x[e];
          v[4 + e] = y[e];
        }
      } else {
#pragma clang loop unroll(full)
        for (int e = 0; e < 8; ++e) v[e] = s[e * st];
      }
      u32x4 h, l;
#pragma clang loop unroll(full)
      for (int e = 0; e < 4; ++e) {
        uint32_t a, b;
        split_pair(v[2 * e], v[2 * e + 1], KIND == kFP16X3 ? 2 : 1, a, b);
        h[e] = a;
        l[e] = b;
      }
      const int row = (mir ? C0 : R0) + i, col = (mir ? R0 : C0) + k;
      if (T > 64 && (row >= np || col >= np)) continue;
      const uint32_t o = plane_off32(row, col, np);
      *reinterpret_cast<u32x4*>(p.hi_out + o) = h;
      if constexpr (KindTraits<KIND>::planes > 1) *reinterpret_cast<u32x4*>(p.lo_out + o) = l;
    }
  }
  if (p.parts_out) {
    t1 = wave_total(t1);
    t2 = 2.0 * wave_total(t2);
    if (lane == 0) {
      red[w] = t1;
      red[kWaveMaxWaves + w] = t2;
    }
    __syncthreads();
    if (t < 2) {
      double s = 0.0;
      for (int k = 0; k < NT / kWave; ++k) s += red[t * kWaveMaxWaves + k];
      p.parts_out[2 * tile + t] = s;
    }
  }
}

// Epilogue of one tile, a 32-row strip at a time.  The waves dump their
// partial rows into LDS transposed ([column][row], four accumulator rows per
// 16-byte write); a thread then sums the partials of four rows of one column
// in piece order, applies v = alpha acc + beta C (+ gamma on the real
// diagonal), stores the FP32 result, adds the traces and leaves v in the image
// (a diagonal tile takes its upper elements and writes each to both places, so
// its image is exactly symmetric).  C was loaded before the K loop: a load
// waits for every store issued before it.  The mirrored FP32 result and the
// planes are written from the image.  The loops stay rolled: code that runs
// once per work-group costs its instruction fetch, about a cycle per byte.
template <int KIND, int MB, int Q>
__device__ __forceinline__ void wave_epilogue(const f32x16 (&acc)[MB][MB],
                                              const f32x4 (&cs)[MB][Q], const Epi& p,
                                              float as, float beta, float gamma, int R0, int C0,
                                              int w, int nw, int lane, float* lds, double* red,
                                              int tile) {
  using Sh = WaveShape<MB>;
  constexpr int T = Sh::T, S = Sh::LD, SP = Sh::LP;
  const int np = p.np, nv = p.n_valid, NT = blockDim.x;
  const bool diag = R0 == C0, use_c = beta != 0.0f;
  const int t = threadIdx.x;
  float* img = lds;               // [column][S]
  float* part = lds + Sh::kImg;   // [wave][column][SP]
  const float oc = (p.centring & kCentredOut) ? kPlaneCentre : 0.0f;
  double t1 = 0.0, t2 = 0.0;
#pragma clang loop unroll(disable)
  for (int mi = 0; mi < MB; ++mi) {
    f32x4 cv[Q];
    float* mine = part + (w * T + (lane & 31)) * SP + 4 * (lane >> 5);
#pragma clang loop unroll(full)
    for (int m = 0; m < MB; ++m) {   // the strip's registers
      if (mi != m) continue;
#pragma clang loop unroll(full)
      for (int i = 0; i < Q; ++i) cv[i] = cs[m][i];
#pragma clang loop unroll(full)
      for (int ni = 0; ni < MB; ++ni)
#pragma clang loop unroll(full)
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(mine + ni * 32 * SP + 8 * q) =
              f32x4{acc[m][ni][4 * q], acc[m][ni][4 * q + 1], acc[m][ni][4 * q + 2],
                    acc[m][ni][4 * q + 3]};
    }
    __syncthreads();
    f32x4 v[Q];
#pragma clang loop unroll(full)
    for (int i = 0; i < Q; ++i) {
      const int q = t + NT * i, c = q % T, r4 = q / T * 4;
      if (q >= 8 * T) break;
      const float* src = part + c * SP + r4;
      v[i] = *reinterpret_cast<const f32x4*>(src);
#pragma clang loop unroll_count(2)
      for (int k = 1; k < nw; ++k) v[i] += *reinterpret_cast<const f32x4*>(src + k * T * SP);
#pragma clang loop unroll(full)
      for (int e = 0; e < 4; ++e)
        v[i][e] = use_c ? fmaf(as, v[i][e], beta * cv[i][e]) : as * v[i][e];
      // rows and columns past np are none (their operands were other rows')
      if (MB > 2 && (R0 + 32 * mi + r4 >= np || C0 + c >= np)) v[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma clang loop unroll(full)
    for (int i = 0; i < Q; ++i) {
      const int q = t + NT * i, c = q % T, r = 32 * mi + q / T * 4;
      const int row = R0 + r, col = C0 + c;
      if (q >= 8 * T) break;
      float* o = p.out + int64_t(row) * p.ld_out + col;
      if (!diag) {
#pragma clang loop unroll(full)
        for (int e = 0; e < 4; ++e) {
          img[c * S + r + e] = v[i][e];
          const double d = static_cast<double>(v[i][e]);
          t2 += d * d;   // each unordered pair counted once: doubled below
          if (p.out && row + e < nv && col < nv) o[int64_t(e) * p.ld_out] = v[i][e];
        }
      } else {
#pragma clang loop unroll(full)
        for (int e = 0; e < 4; ++e) {
          float x = v[i][e];
          const bool on = row + e == col, real_on = on && col < p.n_diag;
          if (row + e <= col) {   // below the diagonal: mirrored from above
            if (real_on) x += gamma;
            img[c * S + r + e] = real_on ? x - oc : x;
            if (!on) img[(r + e) * S + c] = x;
            const double d = static_cast<double>(x);
            t1 += on ? d : 0.0;
            t2 += (on ? 0.5 : 1.0) * d * d;
            if (p.out && col < nv) o[int64_t(e) * p.ld_out] = x;
          }
        }
      }
    }
    __syncthreads();
  }
  tile_finish<KIND, T, S, 1>(p, R0, C0, w, lane, img, red, tile, t1, t2);
}

// The tile of this work-group: nw K pieces of an np-wide K range (linear over
// the segments), one per wave.
template <int KIND, int MB, int NSEG = 1>
__global__ __launch_bounds__(WaveShape<MB>::kMaxWaves * kWave)
__attribute__((amdgpu_waves_per_eu(WaveShape<MB>::kMaxWaves / 4, WaveShape<MB>::kMaxWaves / 4)))
void k_sym_wave(WaveArgs p) {
  using Sh = WaveShape<MB>;
  // K steps held in registers: 32-row tiles load a whole piece of 8 at once
  // (one memory latency per product; half with two segments, which would
  // spill), 64-row ones run a step ahead
  constexpr int NP = KindTraits<KIND>::planes, ST = MB > 1 ? 2 : NSEG == 1 ? 8 : 4;
  constexpr int kLoads = 2 * NP * MB, kMfma = KindTraits<KIND>::products * MB * MB;
  constexpr int kPer = kMfma / kLoads > 0 ? kMfma / kLoads : 1;
  __shared__ __attribute__((aligned(16))) float lds[Sh::kLds];
  __shared__ double red[2 * kWaveMaxWaves];
  const int lane = threadIdx.x & (kWave - 1), nw = p.g.nw;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int np = p.epi.np, lim = p.g.lim;
  const int tile = xcd_remap(blockIdx.x, p.g.ntiles);
  int ti, tj;
  tile_of(tile, p.g.nt, p.g.band, ti, tj);
  const int R0 = ti * Sh::T, C0 = tj * Sh::T;   // R0 <= C0

  // Byte offset of a block at K step 0, and in it of this lane's 16 bytes (row
  // lane % 32, column chunk lane / 32).
  const uint32_t panel = static_cast<uint32_t>(np) * 512;   // bytes of a 256-row panel of one plane
  const uint32_t lo = (lane & 31) * 16 + (lane >> 5) * 4096;
  uint32_t oa[MB], ob[MB];
#pragma clang loop unroll(full)
  for (int i = 0; i < MB; ++i) {
    // (96-row tiles may end past np: those blocks take the last one's rows)
    const int ra = min(R0 / 32 + i, np / 32 - 1), rb = min(C0 / 32 + i, np / 32 - 1);
    oa[i] = (ra >> 3) * panel + (ra & 7) * 512;
    ob[i] = (rb >> 3) * panel + (rb & 7) * 512;
  }
  f32x16 acc[MB][MB];
#pragma clang loop unroll(full)
  for (int mi = 0; mi < MB; ++mi)
#pragma clang loop unroll(full)
    for (int ni = 0; ni < MB; ++ni)
#pragma clang loop unroll(full)
      for (int q = 0; q < 16; ++q) acc[mi][ni][q] = 0.0f;

  // This wave's piece in 16-wide K steps (split_tail's pieces, units of two
  // steps), and its part of a segment: steps past lim would only add zeros.
  const int kseg = np / 16, k2 = NSEG * kseg / 2;
  const int p0 = k2 * w / nw * 2, p1 = k2 * (w + 1) / nw * 2;
  // (a column past lim: both operands' rows are zero)
  const int kend = C0 < lim && w < nw ? lim / 16 : 0;
  auto range = [&](int seg, int& s0, int& s1) {
    s0 = min(max(p0 - seg * kseg, 0), kend);
    s1 = max(min(p1 - seg * kseg, kend), s0);
  };
  WaveFrag<KIND, MB> f[ST];
  auto load = [&](WaveFrag<KIND, MB>& g, int seg, int s) {
    const int64_t ko = int64_t(s) * 8192;
#pragma clang loop unroll(full)
    for (int q = 0; q < NP; ++q) {
      const char* pa = reinterpret_cast<const char*>(p.a[seg][q]) + ko;
      const char* pb = reinterpret_cast<const char*>(p.b[seg][q]) + ko;
#pragma clang loop unroll(full)
      for (int i = 0; i < MB; ++i) {
        g.a[q][i] = *reinterpret_cast<const u32x4*>(pa + oa[i] + lo);
        g.b[q][i] = *reinterpret_cast<const u32x4*>(pb + ob[i] + lo);
      }
    }
  };
  constexpr int kAhead = MB == 1 ? ST : ST - 1;   // steps loaded before the first product
  auto preload = [&](int seg, int s0, int s1) {
#pragma clang loop unroll(full)
    for (int i = 0; i < kAhead; ++i) load(f[i], seg, max(min(s0 + i, s1 - 1), 0));
  };
  int s0, s1;
  range(0, s0, s1);
  if (s1 > s0) preload(0, s0, s1);

  f32x4 cs[MB][Sh::Q];
  constexpr bool kEarlyC = MB * NSEG < 3 || MB == 1;   // else no registers are left for it
  if constexpr (kEarlyC)
#pragma clang loop unroll(full)
    for (int mi = 0; mi < MB; ++mi) wave_load_c<MB>(cs[mi], p.epi, R0, C0, mi);

  const LayerCoef cf = decide_layer_wave(p.dec);
  if (cf.sign == 0) return;
  float alpha = p.epi.alpha, beta = p.epi.beta, gamma = p.epi.gamma;
  if (p.dec.mode != 0) {
    const int cn = p.epi.centring;
    alpha = cf.a;
    beta = (cn & (kCentredSquare | kCentredPair)) ? cf.b + 2.0f * kPlaneCentre * cf.a : cf.b;
    gamma = (cn & kCentredSquare) ? cf.c - kPlaneCentre * kPlaneCentre * cf.a : cf.c;
  }
  // Nothing but the fragments' own loads may be in flight in the K loop: a
  // load of the decision still pending on some path would make the compiler
  // drain the queue wherever its register is reused.
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)

#pragma clang loop unroll(disable)
  for (int seg = 0; seg < NSEG; ++seg) {
    if (seg > 0) {
      range(seg, s0, s1);
      if (s1 > s0) preload(seg, s0, s1);
    }
    if constexpr (MB == 1) {
      // a longer piece comes ST steps at a time
      for (int s = s0; s < s1; s += ST) {
        if (s > s0) preload(seg, s, s1);
#pragma clang loop unroll(full)
        for (int u = 0; u < ST; ++u)
          if (s + u < s1) wave_products<KIND, MB>(f[u], acc);
      }
    } else {
      // step s + u from stage u while the next step loads, one load after
      // every kPer MFMAs (clamped to the range at its end)
      for (int s = s0; s < s1; s += ST) {
#pragma clang loop unroll(full)
        for (int u = 0; u < ST; ++u) {
          __builtin_amdgcn_sched_barrier(0);
          load(f[(u + ST - 1) % ST], seg, min(s + u + ST - 1, s1 - 1));
          wave_products<KIND, MB>(f[u], acc);
#pragma clang loop unroll(full)
          for (int q = 0; q < kLoads; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, kPer, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
  if constexpr (!kEarlyC)
#pragma clang loop unroll(full)
    for (int mi = 0; mi < MB; ++mi) wave_load_c<MB>(cs[mi], p.epi, R0, C0, mi);
  wave_epilogue<KIND, MB>(acc, cs, p.epi, alpha * p.epi.oscale, beta, gamma, R0, C0, w, nw, lane, lds,
                          red, tile);
}

// ---------------------------------------------------------------------------
// Split products on 192 x 192 tiles: the scheme of k_sym_split (four waves,
// here of 96 x 96; LDS ring of K steps filled by copies, fragments double
// buffered in registers, one barrier per step) for orders whose 256 x 256
// tiles, unsplit, would use little more than half the machine.  Wave w copies
// plane w of a step (A hi, A lo, B hi, B lo; 64 rows of one 8-column chunk per
// copy).  The K order is that of k_sym_split, so results are the same bit for
// bit.  C is loaded during the last K steps (the accumulators leave 512 - 240
// registers for it): behind the K loop, in batches with the stores between,
// it took 31 us instead of 6.  The finished values go through an FP32 image of
// the whole tile in LDS ([row][196]: rows are read in 16-byte pieces, columns by
// consecutive lanes, both without bank conflicts).
//
// A layer of n = 4092 takes 197 us against 254.5 us on 136 tiles of 256 x 256:
// 167 us of K loop, which runs at 93% of the MFMA rate of a clock that the power
// limit holds at 1.4 GHz (1340 TFLOP/s over the padded tiles, what a large
// library product reaches), 17 us of epilogue at some 4 TB/s, and the launch.
// ---------------------------------------------------------------------------
constexpr int kMidRows = 192;

template <int KIND, int NSEG = 1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_sym_mid(WaveArgs p) {
  constexpr int T = kMidRows, S = T + 4, NS = 4, M = 3;   // image [row][S]
  constexpr bool kLo = KIND != kBF16X1;
  constexpr int kPlane = T * 32, kSlot = (kLo ? 4 : 2) * kPlane;   // bytes per K step
  constexpr int kCopies = kLo ? 6 : 3;                             // per wave and K step
  __shared__ __attribute__((aligned(1024))) float lds[T * S];
  static_assert(NS * kSlot <= int(sizeof(lds)), "ring exceeds the image");
  __shared__ double red[2 * kWaveMaxWaves];
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int np = p.epi.np, KT = np / 16, ke = NSEG * KT;
  const int tile = xcd_remap(blockIdx.x, p.g.ntiles);
  int ti, tj;
  tile_of(tile, p.g.nt, p.g.band, ti, tj);
  const int R0 = ti * T, C0 = tj * T;

  // This wave's copies of a K step: chunk h, row group g of plane pl (tiles may
  // end past np: those groups take the last rows).
  const int pl = kLo ? w : w >> 1;   // kLo: A hi, A lo, B hi, B lo; else A, B
  const bool isb = kLo ? pl >= 2 : pl == 1;
  const int q = kLo ? pl & 1 : 0;
  uint32_t go[3];
#pragma clang loop unroll(full)
  for (int g = 0; g < 3; ++g) {
    const int row = min((isb ? C0 : R0) + 64 * g, np - 64);
    go[g] = uint32_t(row >> 8) * uint32_t(np) * 512u + (row & 255) * 16u;
  }
  const uint32_t lds0 = static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)(lds)));
  const uint32_t v0 = lane * 16;
  const uint16_t* seg0 = isb ? (q ? p.b[0][1] : p.b[0][0]) : (q ? p.a[0][1] : p.a[0][0]);
  const uint16_t* seg1 = isb ? (q ? p.b[1][1] : p.b[1][0]) : (q ? p.a[1][1] : p.a[1][0]);
  auto source = [&](int k) {
    const bool sg = NSEG == 2 && k >= KT;
    return reinterpret_cast<const char*>(sg ? seg1 : seg0) + int64_t(sg ? k - KT : k) * 8192;
  };
  auto copy = [&](const char* src, int slot, int i) {   // copy i of a K step
    const int h = kLo ? i / 3 : w & 1, g = kLo ? i % 3 : i;
    dma_chunk(v0 + h * 4096, src + go[g], lds0 + slot * kSlot + pl * kPlane + (h * 3 + g) * 1024);
  };
#pragma clang loop unroll(full)
  for (int k = 0; k < NS; ++k) {
    const char* src = source(min(k, ke - 1));
#pragma clang loop unroll(full)
    for (int i = 0; i < kCopies; ++i) copy(src, k, i);
  }

  const LayerCoef cf = decide_layer_wave(p.dec);
  float alpha = p.epi.alpha, beta = p.epi.beta, gamma = p.epi.gamma;
  if (p.dec.mode != 0) {
    const int cn = p.epi.centring;
    alpha = cf.a;
    beta = (cn & (kCentredSquare | kCentredPair)) ? cf.b + 2.0f * kPlaneCentre * cf.a : cf.b;
    gamma = (cn & kCentredSquare) ? cf.c - kPlaneCentre * kPlaneCentre * cf.a : cf.c;
  }
  // the decision's loads, and with them the first copies (a wait that the
  // compiler knows, or it would wait for a register of the decision in the loop)
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  if (cf.sign == 0) return;
  __syncthreads();

  f32x16 acc[M][M];
#pragma clang loop unroll(full)
  for (int mi = 0; mi < M; ++mi)
#pragma clang loop unroll(full)
    for (int ni = 0; ni < M; ++ni)
#pragma clang loop unroll(full)
      for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 0.0f;
  const int wm = w >> 1, wn = w & 1, r = lane & 31, h = lane >> 5;
  const int fa = h * 3072 + (wm * 96 + r) * 16;
  const int fb = (kLo ? 2 : 1) * kPlane + h * 3072 + (wn * 96 + r) * 16;
  const char* ring = reinterpret_cast<const char*>(lds);
  using Frag = WaveFrag<KIND, M>;
  constexpr int kReads = 2 * KindTraits<KIND>::planes * M;
  auto read = [&](Frag& f, int slot, int i) {   // fragment i of a K step
    const char* sl = ring + slot * kSlot + (i / (2 * M)) * kPlane + (i % M) * 512;
    if (i % (2 * M) < M)
      f.a[i / (2 * M)][i % M] = *reinterpret_cast<const u32x4*>(sl + fa);
    else
      f.b[i / (2 * M)][i % M] = *reinterpret_cast<const u32x4*>(sl + fb);
  };
  // Step k from cur while step k + 1 is read into nxt, a read after each of the
  // first MFMAs; before the last NS steps slot k takes step k + NS, a copy after
  // each of the next MFMAs.
  auto products = [&](const Frag& cur, Frag& nxt, int k, bool refill) {
    const char* src = source(k + NS);
    constexpr int pa[3] = {0, 0, 1}, pb[3] = {0, 1, 0};   // hi hi, hi lo, lo hi
    __syncthreads();
#pragma clang loop unroll(full)
    for (int j = 0; j < KindTraits<KIND>::products * M * M; ++j) {
      const int u = j / (M * M), mi = j / M % M, ni = j % M;
      mfma_32x32x16<KIND>(acc[mi][ni], cur.a[pa[u]][mi], cur.b[pb[u]][ni]);
      if (j < kReads) read(nxt, (k + 1) & (NS - 1), j);
      else if (refill && j - kReads < kCopies) copy(src, k & (NS - 1), j - kReads);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto step = [&](const Frag& cur, Frag& nxt, int k) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * kCopies) : "memory");
    products(cur, nxt, k, true);
  };
  auto last_step = [&](const Frag& cur, Frag& nxt, int k) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    products(cur, nxt, k, false);
  };
  Frag f0, f1;
#pragma clang loop unroll(full)
  for (int i = 0; i < kReads; ++i) read(f0, 0, i);
#pragma clang loop unroll(disable)
  for (int k = 0; k < ke - NS; k += 2) {
    step(f0, f1, k);
    step(f1, f0, k + 1);
  }
  // The last NS steps, all copied, with C on its way: four columns of one row
  // per load (a launch without C reads one row of A instead).
  wait_vmem_all();
  // Block (i, j): rows 16 i + 4 w + lane / 16, columns 64 j + 4 (lane % 16).
  const Epi& ep = p.epi;
  const bool diag = R0 == C0, use_c = beta != 0.0f && ep.c;
  const int er = 4 * w + (lane >> 4), ec = (lane & 15) * 4;
  const float* cb = use_c ? ep.c : reinterpret_cast<const float*>(p.a[0][0]);
  const uint32_t cof = use_c ? uint32_t(er) * np + ec : ec;
  f32x4 c[T / 16][3];
#pragma clang loop unroll(full)
  for (int i = 0; i < T / 16; ++i)
#pragma clang loop unroll(full)
    for (int j = 0; j < 3; ++j) {
      const float* blk = cb + (use_c ? int64_t(min(R0 + 16 * i, np - 16)) * np : 0) +
                         min(C0 + 64 * j, np - 64);
      c[i][j] = *reinterpret_cast<const f32x4*>(blk + cof);
    }
  __builtin_amdgcn_sched_barrier(0);
#pragma clang loop unroll(full)
  for (int k = 0; k < NS; k += 2) {
    last_step(f0, f1, ke - NS + k);
    last_step(f1, f0, ke - NS + k + 1);
  }
  __syncthreads();

#pragma clang loop unroll(full)
  for (int mi = 0; mi < M; ++mi)
#pragma clang loop unroll(full)
    for (int ni = 0; ni < M; ++ni)
#pragma clang loop unroll(full)
      for (int e = 0; e < 16; ++e)
        lds[(wm * 96 + mi * 32 + 8 * (e / 4) + 4 * h + e % 4) * S + wn * 96 + ni * 32 + r] =
            acc[mi][ni][e];
  __syncthreads();
  const float as = alpha * ep.oscale, oc = (ep.centring & kCentredOut) ? kPlaneCentre : 0.0f;
  const int nv = ep.n_valid;
  double t1 = 0.0, t2 = 0.0;
  float* img = lds + er * S + ec;
  const int64_t oof = int64_t(er) * ep.ld_out + ec;
#pragma clang loop unroll(full)
  for (int i = 0; i < T / 16; ++i)
#pragma clang loop unroll(full)
    for (int j = 0; j < 3; ++j) {
      const int row0 = R0 + 16 * i, col0 = C0 + 64 * j;
      float* m = img + 16 * i * S + 64 * j;
      f32x4 v = *reinterpret_cast<const f32x4*>(m);
#pragma clang loop unroll(full)
      for (int e = 0; e < 4; ++e) v[e] = use_c ? fmaf(as, v[e], beta * c[i][j][e]) : as * v[e];
      if (row0 >= np || col0 >= np) v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};   // other rows' products
      *reinterpret_cast<f32x4*>(m) = v;
      if (diag && 64 * j + ec <= 16 * i + er) continue;   // left to the next pass
#pragma clang loop unroll(full)
      for (int e = 0; e < 4; ++e) {
        const double d = static_cast<double>(v[e]);
        t2 += d * d;   // doubled in tile_finish
      }
      if (ep.out && ep.vec_ok && row0 + 16 <= nv && col0 + 64 <= nv)
        *reinterpret_cast<f32x4*>(ep.out + int64_t(row0) * ep.ld_out + col0 + oof) = v;
    }
  if (ep.out && !(ep.vec_ok && R0 + T <= nv && C0 + T <= nv)) {
    // blocks that end past the result, or all of an unaligned one
#pragma clang loop unroll(disable)
    for (int b = 0; b < T / 16 * 3; ++b) {
      const int row0 = R0 + b / 3 * 16, col0 = C0 + b % 3 * 64;
      if (ep.vec_ok && row0 + 16 <= nv && col0 + 64 <= nv) continue;
      if (diag && col0 + ec <= row0 + er) continue;
#pragma clang loop unroll(disable)
      for (int e = 0; e < 4; ++e)
        if (row0 + er < nv && col0 + ec + e < nv)
          ep.out[int64_t(row0) * ep.ld_out + col0 + oof + e] = img[b / 3 * 16 * S + b % 3 * 64 + e];
    }
  }
  __syncthreads();
  if (diag) {
    // The groups above the diagonal are mirrored in the image; those on it
    // finish their upper elements.
#pragma clang loop unroll_count(2)
    for (int g = threadIdx.x; g < T * T / 4; g += 256) {
      const int rl = g % T, cl = g / T * 4;   // consecutive rows: no bank conflicts
      if (cl > rl) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(lds + rl * S + cl);
#pragma clang loop unroll(full)
        for (int e = 0; e < 4; ++e) lds[(cl + e) * S + rl] = v[e];
      } else if (cl + 3 >= rl) {
#pragma clang loop unroll(disable)
        for (int e = rl - cl; e < 4; ++e) {
          const int row = R0 + rl, col = C0 + cl + e;
          float x = lds[rl * S + cl + e];
          const bool on = col == row, real_on = on && col < ep.n_diag;
          if (real_on) x += gamma;
          lds[(cl + e) * S + rl] = real_on ? x - oc : x;
          const double d = static_cast<double>(x);
          t1 += on ? d : 0.0;
          t2 += (on ? 0.5 : 1.0) * d * d;
          if (ep.out && col < nv) ep.out[int64_t(row) * ep.ld_out + col] = x;
        }
      }
    }
    __syncthreads();
  }
  tile_finish<KIND, T, 1, S>(ep, R0, C0, w, lane, lds, red, tile, t1, t2);
}

// ---------------------------------------------------------------------------
// FP32 products of small orders, sum_s A_s B_s^T over up to four K segments
// (row-major operands), on the FP32 matrix cores.  Tiles and epilogue as in
// k_sym_wave; eight waves (four for 96-row tiles) take an equal share of the K
// steps (16 values) each.  A wave copies its own blocks (32 rows x 16 values, 64
// contiguous bytes per row) into a private LDS ring with global_load_lds, NS steps
// ahead and without barriers; lane (r, h) reads its eight values of row r, two
// 16-byte pieces at positions swizzled by the row so that eight consecutive rows
// use all banks, half a step ahead into registers, and feeds value 8 h + e to MFMA e.
// A sum is cut after two steps (eight in 96-row tiles): it is added to a second set
// of accumulators and the next begins at zero, so that few roundings meet the
// full size of a result.
//
// Against the 256 x 256 tiles and their split-K kernel: a layer of n = 1026 takes 53
// us (80), n = 1536 89 (90), n = 1792 96 (116), n = 2046 120 (145); an FP32 solve of n
// = 256 345 us (1039).  Of the 28 us of the product at n = 1026, 18 are the K loop, at
// 80% of the FP32 matrix-core rate, 10 the launch, the decision and the epilogue.
// Relative error of a layer of n = 1536 1.2e-7 (2.2e-7), n = 2046 2.2e-7 (3.3e-7), of
// an FP32 solve of n = 1026 3.4e-7 (5.5e-7).
// ---------------------------------------------------------------------------

struct WaveF32Args {
  const float* a[4];
  const float* b[4];
  Epi epi;
  Decide dec;
  WaveGrid g;
};

// Waves of a work-group: two per SIMD, one where a wave's two sets of
// accumulators of 96 rows and two K steps take more than half the registers.
template <int MB>
constexpr int kWaveF32Waves = MB < 3 ? 8 : 4;
// K steps (16 values) summed in one set of accumulators.
template <int MB>
constexpr int kF32Cut = MB < 3 ? 2 : 8;   // (one wave per SIMD: nothing hides the additions)

template <int MB, int NSEG>
__global__ __launch_bounds__(kWaveF32Waves<MB> * kWave)
__attribute__((amdgpu_waves_per_eu(kWaveF32Waves<MB> / 4, kWaveF32Waves<MB> / 4)))
void k_wave_f32(WaveF32Args p) {
  using Sh = WaveShape<MB>;
  constexpr int NW = kWaveF32Waves<MB>, NS = MB == 1 ? 4 : 2;   // ring slots per wave
  constexpr int kSlot = MB * 2 * 2048;                      // bytes: A blocks, B blocks
  constexpr int kCopies = MB * 2 * 2;                       // 1 KB copies per step
  static_assert((Sh::kImg + NW * Sh::T * Sh::LP) * 4 <= NW * NS * kSlot, "epilogue fits the ring");
  __shared__ __attribute__((aligned(1024))) float lds[NW * NS * kSlot / 4];
  __shared__ double red[2 * kWaveMaxWaves];
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int np = p.epi.np, lim = p.g.lim;
  const int tile = xcd_remap(blockIdx.x, p.g.ntiles);
  int ti, tj;
  tile_of(tile, p.g.nt, p.g.band, ti, tj);
  const int R0 = ti * Sh::T, C0 = tj * Sh::T;   // R0 <= C0

  // This wave's K steps [s0, s0 + qn) of those of all segments together (a column
  // past lim: both operands' rows are zero).
  const int ks = C0 < lim ? lim / 16 : 0;
  const int s0 = NSEG * ks * w / NW, qn = NSEG * ks * (w + 1) / NW - s0;
  // Copy i of a block: rows 16 i + lane / 4, 16-byte piece (lane % 4) of the
  // row's 64 bytes, which holds values 4 c .. 4 c + 3 with
  // c = (lane % 4) ^ (row / 2 % 4).
  const uint32_t src = ((lane & 3) ^ ((lane >> 3) & 3)) * 16;
  const uint32_t own = uint32_t(lane >> 2) * np * 4u + src;
  const uint32_t ring0 =
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)(lds))) +
      w * (NS * kSlot);
  struct Source {
    const float *a, *b;
  };
  auto source = [&](int q) {   // step q
    int x = s0 + q;
    const int sg = (NSEG > 1 && x >= ks) + (NSEG > 2 && x >= 2 * ks) + (NSEG > 2 && x >= 3 * ks);
    x -= sg * ks;
    return Source{(sg == 0 ? p.a[0] : sg == 1 ? p.a[1] : sg == 2 ? p.a[2] : p.a[3]) + x * 16,
                  (sg == 0 ? p.b[0] : sg == 1 ? p.b[1] : sg == 2 ? p.b[2] : p.b[3]) + x * 16};
  };
  // Copy c of step q into its slot: half u of block i of an operand (96-row tiles
  // may end past np: those blocks take the last one's rows).
  auto copy = [&](const Source& g, int q, int c) {
    const int i = c / 4, u = c / 2 % 2, isb = c % 2;
    const float* rows = (isb ? g.b : g.a) +
                        (int64_t(min((isb ? C0 : R0) + 32 * i, np - 32)) + u * 16) * np;
    dma_chunk(own, rows, ring0 + (q & (NS - 1)) * kSlot + (isb * MB + i) * 2048 + u * 1024);
  };
#pragma clang loop unroll(full)
  for (int i = 0; i < NS; ++i)
    if (i < qn) {
      const Source g = source(i);
#pragma clang loop unroll(full)
      for (int c = 0; c < kCopies; ++c) copy(g, i, c);
    }

  const LayerCoef cf = decide_layer_wave(p.dec);
  float alpha = p.epi.alpha, beta = p.epi.beta, gamma = p.epi.gamma;
  if (p.dec.mode != 0) {
    alpha = cf.a;
    beta = cf.b;
    gamma = cf.c;
  }
  f32x16 acc[MB][MB], sum[MB][MB];
#pragma clang loop unroll(full)
  for (int mi = 0; mi < MB; ++mi)
#pragma clang loop unroll(full)
    for (int ni = 0; ni < MB; ++ni)
#pragma clang loop unroll(full)
      for (int q = 0; q < 16; ++q) sum[mi][ni][q] = 0.0f;
  // this lane's two 16-byte pieces of its row (values 8 h .. 8 h + 7) in a block
  const int r = lane & 31, h2 = (lane >> 5) * 2;
  const int f0 = r * 64 + ((h2 ^ ((r >> 1) & 3)) * 16), f1 = r * 64 + (((h2 + 1) ^ ((r >> 1) & 3)) * 16);
  const char* ring = reinterpret_cast<const char*>(lds) + w * (NS * kSlot);
  wait_vmem_all();   // the decision's loads, and with them the first copies
  if (cf.sign == 0) return;

  struct Frag {   // half a step: one of the two pieces of every block
    f32x4 a[MB], b[MB];
  };
  auto read = [&](Frag& f, int q, int off) {
    const char* sl = ring + (q & (NS - 1)) * kSlot + off;
#pragma clang loop unroll(full)
    for (int i = 0; i < MB; ++i) {
      f.a[i] = *reinterpret_cast<const f32x4*>(sl + i * 2048);
      f.b[i] = *reinterpret_cast<const f32x4*>(sl + (MB + i) * 2048);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Four products of every pair of blocks, half a step; first: of a new sum.
  auto products = [&](const Frag& f, auto first) {
#pragma clang loop unroll(full)
    for (int e = 0; e < 4; ++e)
#pragma clang loop unroll(full)
      for (int mi = 0; mi < MB; ++mi)
#pragma clang loop unroll(full)
        for (int ni = 0; ni < MB; ++ni) {
          if (decltype(first)::value && e == 0) {
#pragma clang loop unroll(full)
            for (int k = 0; k < 16; ++k) acc[mi][ni][k] = 0.0f;
          }
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[mi][e], f.b[ni][e], acc[mi][ni], 0, 0, 0);
        }
    __builtin_amdgcn_sched_barrier(0);
  };
  Frag x, y;
  read(x, 0, f0);
  auto step = [&](int q, auto first) {
    read(y, q, f1);
    products(x, first);
    // The reads of step q are done: its slot takes step q + NS.  Step q + 1 has
    // arrived once no more than the copies after it are outstanding (at the end a
    // slot that no step fills any more is read, and not used).
    if (q + NS < qn) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      const Source g = source(q + NS);
#pragma clang loop unroll(full)
      for (int c = 0; c < kCopies; ++c) copy(g, q, c);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * kCopies) : "memory");
    } else {
      wait_vmem_all();
    }
    read(x, q + 1, f0);
    products(y, std::false_type());
  };
#pragma clang loop unroll(disable)
  for (int q = 0; q < qn;) {
    const int qe = min(q + kF32Cut<MB>, qn);
    step(q, std::true_type());
#pragma clang loop unroll(disable)
    while (++q < qe) step(q, std::false_type());
#pragma clang loop unroll(full)
    for (int mi = 0; mi < MB; ++mi)
#pragma clang loop unroll(full)
      for (int ni = 0; ni < MB; ++ni)
#pragma clang loop unroll(full)
        for (int k = 0; k < 16; ++k) sum[mi][ni][k] += acc[mi][ni][k];
  }
  f32x4 cs[MB][Sh::groups(NW)];
#pragma clang loop unroll(full)
  for (int mi = 0; mi < MB; ++mi) wave_load_c<MB>(cs[mi], p.epi, R0, C0, mi);
  wait_vmem_all();
  __syncthreads();   // the rings are free
  wave_epilogue<kF32, MB>(sum, cs, p.epi, alpha * p.epi.oscale, beta, gamma, R0, C0, w, NW, lane, lds,
                          red, tile);
}

}  // namespace sp2
