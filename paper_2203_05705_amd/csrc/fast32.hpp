// fp32 products for gfx950: matrix-core kernels whose fragments come straight from memory.
//
// v_mfma_f32_16x16x4_f32 runs at a sixteenth of the bf16 rate (154 TFLOP/s measured for a large library
// product), so an fp32 product is bound by the matrix cores long before LDS or the L1 matter: a wavefront
// tile of 64 x 64 needs 16 bytes per clock and CU.  The operands therefore skip LDS altogether: every lane
// loads the elements its MFMAs take, 4 contraction indices of a row at a time, D steps of 16 ahead, and the
// index maps of a row pattern (any affine map of rows, columns and contraction, lists of rows, tile-class
// block progressions) cost nothing but a different loop-invariant lane offset.  No operand has to be aligned
// or padded: loads are dword-aligned, only the last partial step of a contraction tests its indices.
//   KC operand (element (row, k) at p[row*ld + k]): lane (i = l%16, g = l/16) loads k = 4g .. 4g+3 of row
//     16t + i of every 16-row tile t, one 16-byte load (VEC) or, when the contraction map is strided, four.
//   MC operand (element (row, k) at p[k*ld + row]): for each of k = 4g .. 4g+3 the T rows T*i .. T*i + T-1,
//     one load of T floats (VEC) or T single ones; tile t of the wavefront is then made of rows T*i + t.
// A workgroup has 256 threads.  What varies is how its four wavefronts share the work: side by side on a
// 128 x 128 tile, or all on the same 64 x 64, 32 x 32 or 16 x 16 tile with the contraction dealt over them
// (small layers: many tiles and short chains instead of few long ones).  The accumulators meet in LDS, where
// they are summed in a fixed order and from where whole rows of the output leave, dropped positions included.
#pragma once
#include "fast.hpp"

namespace ard {

// (What every workgroup reads first comes first: the arguments are fetched line by line.)
struct F32Params {
  const float *A, *B;
  int lda, ldb;
  int M, N, ncls;        // (ncls: tab.ncls, set_bands)
  int splits, tiles_m, tiles_n, group_m, total_tiles;
  FastDiv tiles_div, band_div;           // total_tiles, group_m * tiles_n
  int ka_off, ka_step, kb_off, kb_step;  // affine contraction map of each operand
  Axis am, bn, k;        // plain mode: rows of A, rows of B, contraction (length; maps per operand above)
  const int* kb_cnt;     // (always NULL: direct_assign's per-tile lists are a bf16 feature)
  float* part;           // != NULL: fp32 partial sums part[split][M][N] instead of C
  OutMat C;
  FastDiv row_div, col_div;          // C.rm.step, C.cn.step (affine maps; rows: finishing pass only)
  int c_rows_mapped, c_cols_mapped;  // tile classes: output rows / columns go through the M / N map
  F32Conv cv;
  ClassTab tab;
};

enum { F32_KC_VEC = 0, F32_KC = 1, F32_MC_VEC = 2, F32_MC = 3 };

// floats that are only known to be 4-byte aligned (global memory takes wide loads at any dword)
template <int T> struct __attribute__((packed, aligned(4))) F32Run { float f[T]; };

template <int KIND, int T> struct F32Loader;

template <int KIND, int T> struct F32LoaderKC {
  static constexpr int LOADS = KIND == F32_KC_VEC ? T : 4 * T;  // load instructions per step
  const char* base;
  uint32_t voff[T];
  uint32_t kst;   // bytes between consecutive contraction indices
  int k4;         // first of this lane's four contraction indices within a step
  // `phys`: the physical rows of this wavefront's tile rows (table in LDS; affine axes do without)
  __device__ __forceinline__ void init(const float* p, int ld, const Axis& r, const int* phys, int row0, int lane, int kstep) {
    base = reinterpret_cast<const char*>(p);
    const int i = lane & 15, g = lane >> 4;
    k4 = 4 * g;
    kst = (uint32_t)kstep * 4u;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int row = r.kind == AX_AFFINE ? r.off + imin(row0 + 16 * t + i, r.n - 1) * r.step : phys[16 * t + i];
      voff[t] = ((uint32_t)row * (uint32_t)ld + (uint32_t)(4 * g * kstep)) * 4u;
    }
  }
  // MODE 1, 2: rows are plain, `ld` elements apart
  __device__ __forceinline__ void init_rows(const float* p, int ld, int n, int row0, int lane) {
    base = reinterpret_cast<const char*>(p);
    k4 = 4 * (lane >> 4);
    kst = 4u;
#pragma unroll
    for (int t = 0; t < T; ++t) voff[t] = ((uint32_t)imin(row0 + 16 * t + (lane & 15), n - 1) * (uint32_t)ld + (uint32_t)k4) * 4u;
  }
  // MODE 2: columns = (tap, channel): the channel's plane, shifted by the tap
  __device__ __forceinline__ void init_tap_columns(const float* p, const F32Conv& cv, int ncols, int row0, int lane) {
    base = reinterpret_cast<const char*>(p);
    k4 = 4 * (lane >> 4);
    kst = 4u;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int col = imin(row0 + 16 * t + (lane & 15), ncols - 1);
      const int tap = (int)fdiv((uint32_t)col, cv.by_cp), r = (int)fdiv((uint32_t)tap, cv.by_kw);
      voff[t] = ((uint32_t)(col - tap * cv.Cp) * (uint32_t)cv.plane + (uint32_t)(r * cv.Wg + tap - r * cv.kw + k4)) * 4u;
    }
  }
  __device__ __forceinline__ long slab(int kphys) const { return (long)kphys * 4; }
  __device__ __forceinline__ void load(float (&v)[T][4], long off) const {
    const char* sb = base + off;  // uniform
    if constexpr (KIND == F32_KC_VEC) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const F32Run<4> q = *reinterpret_cast<const F32Run<4>*>(sb + voff[t]);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[t][e] = q.f[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const char* se = sb + (long)e * kst;
#pragma unroll
        for (int t = 0; t < T; ++t) v[t][e] = *reinterpret_cast<const float*>(se + voff[t]);
      }
    }
  }
  // (masks and clamped offsets instead of conditions: the loads of a partial step must not stand behind branches)
  __device__ __forceinline__ void load_tail(float (&v)[T][4], long off, int krem) const {
    const char* sb = base + off;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t m = k4 + e < krem ? ~0u : 0u;
      asm("" : "+v"(m));
#pragma unroll
      for (int t = 0; t < T; ++t)  // beyond the end: the row's first index of the step
        v[t][e] = __uint_as_float(*reinterpret_cast<const uint32_t*>(sb + (voff[t] - (uint32_t)k4 * kst) + (((uint32_t)k4 + e) * kst & m)) & m);
    }
  }
  // row of the workgroup's tile (relative to the wavefront's first row) that MFMA row i of tile t holds
  __device__ __forceinline__ static int local_row(const Axis&, int, int t, int i) { return 16 * t + i; }
};
template <int T> struct F32Loader<F32_KC_VEC, T> : F32LoaderKC<F32_KC_VEC, T> {};
template <int T> struct F32Loader<F32_KC, T> : F32LoaderKC<F32_KC, T> {};

template <int KIND, int T> struct F32LoaderMC {
  static constexpr bool VEC = KIND == F32_MC_VEC;
  static constexpr int NV = VEC ? 1 : T;
  static constexpr int LOADS = 4 * NV;
  const char* base;
  uint32_t voff[NV];
  long kst;       // bytes between consecutive contraction indices
  long kunit;     // bytes per physical contraction index
  int k4;
  // (VEC: the last group of an affine axis is moved back so that it ends with the axis; it then holds rows of
  // the group before as well, computed twice with the same result.  A block axis has extents of whole groups.)
  __device__ __forceinline__ static int group_start(const Axis& r, int row0, int i) {
    return imin(row0 + T * i, r.n - T);
  }
  __device__ __forceinline__ void init(const float* p, int ld, const Axis& r, const int* phys, int row0, int lane, int kstep) {
    base = reinterpret_cast<const char*>(p);
    const int i = lane & 15, g = lane >> 4;
    k4 = 4 * g;
    kunit = (long)ld * 4;
    kst = (long)kstep * ld * 4;
    if constexpr (VEC) {
      // (affine axes are contiguous here; the table holds the group's first row, a moved group lies before it)
      const int prow = r.kind == AX_AFFINE ? r.off + group_start(r, row0, i) : imin(phys[T * i], r.nphys - T);
      voff[0] = ((uint32_t)(4 * g * kstep) * (uint32_t)ld + (uint32_t)prow) * 4u;
    } else {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int row = r.kind == AX_AFFINE ? r.off + imin(row0 + T * i + t, r.n - 1) * r.step : phys[T * i + t];
        voff[t] = ((uint32_t)(4 * g * kstep) * (uint32_t)ld + (uint32_t)row) * 4u;
      }
    }
  }
  // MODE 1: rows = output pixels, contraction = channels of one tap (`plane` elements apart)
  __device__ __forceinline__ void init_pixels(const float* p, const F32Conv& cv, int row0, int lane) {
    base = reinterpret_cast<const char*>(p);
    const int i = lane & 15, g = lane >> 4;
    k4 = 4 * g;
    kunit = kst = (long)cv.plane * 4;
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      // (VEC: output rows are whole groups of T pixels, so a group never straddles two)
      const int row = VEC ? imin(row0 + T * i, cv.npix - T) : imin(row0 + T * i + t, cv.npix - 1);
      const int n = (int)fdiv((uint32_t)row, cv.per_img), rem = row - n * cv.HoWo;
      const int ho = (int)fdiv((uint32_t)rem, cv.per_row), wo = rem - ho * cv.Wo;
      voff[t] = ((uint32_t)(n * cv.Cp + 4 * g) * (uint32_t)cv.plane + (uint32_t)(ho * cv.Wg + wo)) * 4u;
    }
  }
  __device__ __forceinline__ long slab(int kphys) const { return (long)kphys * kunit; }
  __device__ __forceinline__ void load(float (&v)[T][4], long off) const {
    const char* sb = base + off;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const char* se = sb + e * kst;  // uniform
      if constexpr (VEC) {
        const F32Run<T> q = *reinterpret_cast<const F32Run<T>*>(se + voff[0]);
#pragma unroll
        for (int t = 0; t < T; ++t) v[t][e] = q.f[t];
      } else {
#pragma unroll
        for (int t = 0; t < T; ++t) v[t][e] = *reinterpret_cast<const float*>(se + voff[t]);
      }
    }
  }
  __device__ __forceinline__ void load_tail(float (&v)[T][4], long off, int krem) const {
    const char* sb = base + off;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t m = k4 + e < krem ? ~0u : 0u;
      asm("" : "+v"(m));
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const uint32_t o = VEC ? voff[0] + 4u * t : voff[VEC ? 0 : t];
        v[t][e] = __uint_as_float(*reinterpret_cast<const uint32_t*>(sb + (o - (uint32_t)k4 * (uint32_t)kst) + (((uint32_t)k4 + e) * (uint32_t)kst & m)) & m);
      }
    }
  }
  __device__ __forceinline__ static int local_row(const Axis& r, int row0, int t, int i) {
    return VEC ? group_start(r, row0, i) - row0 + t : T * i + t;
  }
};
template <int T> struct F32Loader<F32_MC_VEC, T> : F32LoaderMC<F32_MC_VEC, T> {};
template <int T> struct F32Loader<F32_MC, T> : F32LoaderMC<F32_MC, T> {};

// How many whole 16-deep steps a contraction has, and how many indices its last partial step: a block
// progression counts its last block in full even when the operand ends inside it.
__host__ __device__ __forceinline__ void f32_steps(const Axis& k, int& full, int& rem) {
  int n = k.n;
  if (k.kind == AX_BAFF && n > 0) {
    const int nb = n / k.bs, start = (k.off + (nb - 1) * k.step) * k.bs;
    if (start + k.bs > k.nphys) n = (nb - 1) * k.bs + imax(k.nphys - start, 0);
  }
  full = n >> 4;
  rem = n & 15;
}

// f(std::integral_constant<int, n>) for the n in 1 .. N.
template <int N, class F>
__device__ __forceinline__ void f32_pick(int n, const F& f) {
  if constexpr (N == 1) f(std::integral_constant<int, 1>{});
  else if (n == N) f(std::integral_constant<int, N>{});
  else f32_pick<N - 1>(n, f);
}

// Tile of 16*TM*WM x 16*TN*WN outputs, the contraction dealt over WK groups of wavefronts, D steps in flight.
// MODE 0: plain product.  MODE 1: convolution (A: packed weights, B: pixels of the bordered grid).
// MODE 2: its weight gradient, contraction over the pixels of the grid planes.  Between the output positions lie border
// pixels, where the gradient is zero but the shifted activations are not (they are the next row's or, at a plane's end, the
// next channel's): an infinity or NaN among those would reach sums it has no part in.  Such a term makes its sum NaN, and a
// sum that ends finite had none; a wavefront with any other sum contracts again with the border's elements masked.  (Masks
// in the one loop, 16 v_and for 64 MFMAs, took the gradient of the 32 x 32 layer in conv.hip from 33.6 to 36.5 - 39 us
// wherever they were placed.)
template <int AK, int BK, int TM, int TN, int WM, int WN, int WK, int D, int MODE, bool IN_RUNS>
__device__ __forceinline__ void f32_body(const F32Params& P, const int block_id, float* const lds) {
  constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN, PITCH = BN + 1;
  static_assert(WM * WN * WK == 4, "four wavefronts");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
  touch_args<(MODE == 0 ? 6 : 7)>(P);
  if (MODE == 0 && P.ncls) touch_args<(int)(sizeof(ClassTab) / 64)>(P.tab);
  DirectWork w;
  if (!direct_assign<BM, BN>(P, block_id, w)) return;
  f32x4_t acc[TM][TN];
#pragma unroll
  for (int im = 0; im < TM; ++im)
#pragma unroll
    for (int in = 0; in < TN; ++in)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[im][in][v] = 0.0f;
  const int mrow0 = w.m0 + wm * 16 * TM, nrow0 = w.n0 + wn * 16 * TN;
  // physical rows of the tile's rows of A and of B where they are not affine, looked up once (rows beyond an operand read its last one and
  // are never stored; a block axis counts its last block in full even when the operand ends inside it)
  int* const tab = reinterpret_cast<int*>(lds + WK * BM * PITCH);
  if (MODE == 0 && (w.am.kind != AX_AFFINE || w.bn.kind != AX_AFFINE)) {
    for (int x = tid; x < BM + BN; x += 256) {
      const bool b = x >= BM;
      const Axis& r = b ? w.bn : w.am;
      tab[x] = r.n > 0 ? imin(ax_phys(r, imin((b ? w.n0 - BM : w.m0) + x, r.n - 1)), r.nphys - 1) : 0;
    }
    __syncthreads();
  }
  if (w.kax.n > 0) {
    int full, rem;
    f32_steps(w.kax, full, rem);
    const int all = full + (rem ? 1 : 0);
    const int g_lo = (int)((long)w.split * all / P.splits), g_hi = (int)((long)(w.split + 1) * all / P.splits);
    const int s_lo = g_lo + (int)((long)wk * (g_hi - g_lo) / WK), s_hi = g_lo + (int)((long)(wk + 1) * (g_hi - g_lo) / WK);
    const int e_full = imin(s_hi, full);
    const bool blocks = w.kax.kind == AX_BAFF;
    F32Loader<AK, TM> la;
    F32Loader<BK, TN> lb;
    if constexpr (MODE == 0) {
      la.init(P.A, P.lda, w.am, tab + wm * 16 * TM, mrow0, lane, blocks ? 1 : P.ka_step);
      lb.init(P.B, P.ldb, w.bn, tab + BM + wn * 16 * TN, nrow0, lane, blocks ? 1 : P.kb_step);
    } else {
      // rows of A: channels (MODE 1: rows of the packed weights, MODE 2: planes of the gradient's grid)
      la.init_rows(P.A, P.lda, P.M, mrow0, lane);
      if constexpr (MODE == 1) lb.init_pixels(P.B, P.cv, nrow0, lane);
      else lb.init_tap_columns(P.B, P.cv, P.N, nrow0, lane);
    }
    // Byte offsets of the next step to load; steps are loaded in order, so a step only adds an increment, and
    // after `left` of them (a block of a tile class, a tap, an image) the jump to the next run.
    long oa, ob, inc_a, inc_b, jump_a = 0, jump_b = 0;
    int left = 0x7fffffff, run = 0x7fffffff;
    if constexpr (MODE == 1) {
      const int tap = (int)fdiv((uint32_t)s_lo, P.cv.steps_inner), in_tap = s_lo - tap * (P.cv.Cp >> 4);
      const int r = (int)fdiv((uint32_t)tap, P.cv.by_kw);
      oa = (long)s_lo * 64, inc_a = 64;
      ob = ((long)in_tap * 16 * P.cv.plane + r * P.cv.Wg + tap - r * P.cv.kw) * 4, inc_b = (long)P.cv.plane * 64;
      run = P.cv.Cp >> 4, left = run - in_tap;
    } else if constexpr (MODE == 2) {
      const int n = (int)fdiv((uint32_t)s_lo, P.cv.steps_inner), q = s_lo * 16 - n * P.cv.plane;
      oa = ((long)n * P.cv.Co * P.cv.plane + q) * 4, ob = ((long)n * P.cv.Cp * P.cv.plane + q) * 4;
      inc_a = inc_b = 64;
      run = P.cv.plane >> 4, left = run - (q >> 4);
      jump_a = (long)(P.cv.Co - 1) * P.cv.plane * 4, jump_b = (long)(P.cv.Cp - 1) * P.cv.plane * 4;
    } else if (blocks) {
      const int p = fast_kslab(w.kax, s_lo * 16);
      oa = la.slab(p), ob = lb.slab(p), inc_a = la.slab(16), inc_b = lb.slab(16);
      run = w.kax.bs >> 4, left = run - s_lo % run;
      jump_a = la.slab((w.kax.step - 1) * w.kax.bs), jump_b = lb.slab((w.kax.step - 1) * w.kax.bs);
    } else {
      oa = la.slab(P.ka_off + s_lo * 16 * P.ka_step), ob = lb.slab(P.kb_off + s_lo * 16 * P.kb_step);
      inc_a = la.slab(16 * P.ka_step), inc_b = lb.slab(16 * P.kb_step);
    }
    int tap_r = 0, tap_s = 0;  // MODE 1: where the tap of the next step lies
    if constexpr (MODE == 1) {
      const int tap = (int)fdiv((uint32_t)s_lo, P.cv.steps_inner);
      tap_r = (int)fdiv((uint32_t)tap, P.cv.by_kw), tap_s = tap - tap_r * P.cv.kw;
    }
    auto advance = [&] {
      oa += inc_a, ob += inc_b;
      if (--left == 0) {
        left = run;
        if constexpr (MODE == 1) {
          if (++tap_s == P.cv.kw) tap_s = 0, ++tap_r;
          ob = (long)(tap_r * P.cv.Wg + tap_s) * 4;
        } else {
          oa += jump_a, ob += jump_b;
        }
      }
    };
    const long oa0 = oa, ob0 = ob;
    const int left0 = left;
    float a[D][TM][4], b[D][TN][4];
    const int n_full = e_full - s_lo;
    int ahead = n_full;  // steps still to load
    auto load = [&](int slot) {
      la.load(a[slot], oa);
      lb.load(b[slot], ob);
      if (--ahead > 0) advance();  // (past the end the last step is loaded again: no load stands behind a branch)
    };
    auto mma = [&](const float (&x)[TM][4], const float (&y)[TN][4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int im = 0; im < TM; ++im)
#pragma unroll
          for (int in = 0; in < TN; ++in) acc[im][in] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[im][e], y[in][e], acc[im][in], 0, 0, 0);
    };
    // Step s sits in slot s % D.  Step s + D - 1 is loaded beside the MFMAs of step s, into the slot step s - 1
    // has left.  Every load of a round is unconditional and in order, so that the compiler can count exactly how
    // many younger loads may stay in flight when a step's operands are wanted (with loads behind branches it
    // waited for all of them: a whole memory latency every D steps).
    constexpr int LOADS = F32Loader<AK, TM>::LOADS + F32Loader<BK, TN>::LOADS, MMAS = 4 * TM * TN;
    // Small tiles with operands at 4 bytes a load take a contraction of few steps at once, or in two goes, in code of its
    // own for each number of them, so that this counting still works: the rounds load up to D - 1 steps past the end, which
    // with loads this narrow cost as much as the contraction did (145 x 448 -> 320, strides 3 and 4: forward and data
    // gradient 9.7 -> 5.0 us; 64 x 784 -> 1024, stride 2: data gradient 10.4 -> 7.6, weight gradient 7.7 -> 6.5).  With wide
    // loads it gains nothing (6.0 against 5.8 us) and its code delays the rounds (7.0 -> 7.7 us of 12 steps).  So it does in
    // convolutions, which rarely have so few steps: 9 x 173 channels of 27 x 27 from 384, 3 x 3, data gradient 135 us, with
    // that code 154; 1 x 1 from 96 channels 7.0, with it 6.0.
    auto at_once = [&](auto steps) {
      constexpr int N = decltype(steps)::value;
#pragma unroll
      for (int d = 0; d < N; ++d) load(d);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < N; ++d) mma(a[d], b[d]);
    };
    constexpr bool SCATTERED = AK == F32_KC || BK == F32_KC || AK == F32_MC || BK == F32_MC;
    if (MODE == 0 && SCATTERED && BM * BN <= 1024 && n_full > 0 && n_full <= 2 * D - 2) {
      if (n_full > D) at_once(std::integral_constant<int, D>{});
      f32_pick<D>(n_full > D ? n_full - D : n_full, at_once);
    } else if (n_full > 0) {
#pragma unroll
      for (int d = 0; d < D - 1; ++d) {
        load(d);
        __builtin_amdgcn_sched_barrier(0);
      }
      int s = 0;
      for (; s + D <= n_full; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          load((d + D - 1) % D);
          mma(a[d], b[d]);
          constexpr int PER = MMAS / LOADS > 0 ? MMAS / LOADS : 1;
#pragma unroll
          for (int x = 0; x < LOADS; ++x) {
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // one load,
            __builtin_amdgcn_sched_group_barrier(0x008, PER, 0); // then as many MFMAs as spread the step's loads evenly
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int d = 0; d < D - 1; ++d)
        if (s + d < n_full) mma(a[d], b[d]);
    }
    if constexpr (MODE == 2) {
      float odd[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // stays 0, or becomes NaN
#pragma unroll
      for (int im = 0; im < TM; ++im)
#pragma unroll
        for (int in = 0; in < TN; ++in)
#pragma unroll
          for (int v = 0; v < 4; ++v) odd[v] = __builtin_fmaf(acc[im][in][v], 0.0f, odd[v]);
      if (__any(odd[0] + odd[1] + odd[2] + odd[3] != 0.0f)) {
#pragma unroll
        for (int im = 0; im < TM; ++im)
#pragma unroll
          for (int in = 0; in < TN; ++in)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[im][in][v] = 0.0f;
        oa = oa0, ob = ob0, left = left0;
        for (int s = s_lo; s < e_full; ++s) {
          la.load(a[0], oa);
          lb.load(b[0], ob);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int q = (run - left) * 16 + lb.k4 + e;  // position in the plane
            const bool out = q - (int)fdiv((uint32_t)q, P.cv.per_row) * P.cv.Wg < P.cv.Wo && q < P.cv.npix;
#pragma unroll
            for (int t = 0; t < TN; ++t) b[0][t][e] = out ? b[0][t][e] : 0.0f;
          }
          mma(a[0], b[0]);
          if (s + 1 < e_full) advance();
        }
      }
    }
    if constexpr (MODE == 0) {
      if (rem && s_hi == all && e_full < s_hi) {
        if (n_full > 0) advance();
        la.load_tail(a[0], oa, rem);
        lb.load_tail(b[0], ob, rem);
        mma(a[0], b[0]);
      }
    }
  }
  // A convolution's tile whose wavefronts hold all of their sums: a lane has TN neighbouring pixels of its rows, which leave from the
  // registers (64 rows, 65536 pixels, K = 288: by way of LDS, a float at a time, 33 us, so 29).
  if constexpr (MODE == 1 && BK == F32_MC_VEC && WK == 1) {
    const OutMat& C = P.C;
    if (!C.fill && !C.relu && !C.relu_src && C.beta == 0.0f) {
      const int j = nrow0 + TN * (lane & 15), n = (int)fdiv((uint32_t)imin(j, P.N - TN), P.cv.per_img);  // (planes are whole groups of pixels)
      float* const o = (float*)C.p + (long)n * C.img_stride + (j - n * P.cv.HoWo);
      int r[TM][4];
#pragma unroll
      for (int im = 0; im < TM; ++im)
#pragma unroll
        for (int v = 0; v < 4; ++v) r[im][v] = ax_phys(C.rm, imin(mrow0 + 16 * im + 4 * (lane >> 4) + v, P.M - 1));
      if (j < P.N)
#pragma unroll
        for (int im = 0; im < TM; ++im)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (mrow0 + 16 * im + 4 * (lane >> 4) + v >= P.M) continue;
            F32Run<TN> x;
#pragma unroll
            for (int t = 0; t < TN; ++t) x.f[t] = C.alpha * acc[im][t][v];
            *reinterpret_cast<F32Run<TN>*>(o + (long)r[im][v] * C.plane) = x;
          }
      return;
    }
  }
  // accumulators -> LDS [WK][BM][PITCH]; lane holds column (lane & 15) of a 16 x 16 tile, rows 4*(lane >> 4) + v
  {
    float* mine = lds + wk * BM * PITCH;
#pragma unroll
    for (int in = 0; in < TN; ++in) {
      const int lc = F32Loader<BK, TN>::local_row(w.bn, nrow0, in, lane & 15) + wn * 16 * TN;
#pragma unroll
      for (int im = 0; im < TM; ++im)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int lr = F32Loader<AK, TM>::local_row(w.am, mrow0, im, 4 * (lane >> 4) + v) + wm * 16 * TM;
          if (lr >= 0 && lc >= 0) mine[lr * PITCH + lc] = acc[im][in][v];
        }
    }
  }
  __syncthreads();  // (also: nobody reads the row table any more)
  auto sum = [&](int lr, int lc) {
    float x = lds[lr * PITCH + lc];
#pragma unroll
    for (int k = 1; k < WK; ++k) x += lds[(k * BM + lr) * PITCH + lc];
    return x;
  };
  const OutMat& C = P.C;
  constexpr int CL = BN < 64 ? BN : 64;           // threads along a row of the tile
  constexpr int RP = 256 / CL;
  const int tc = tid % CL, tr = tid / CL;
  // One loop for every kind of output: a slot of the tile's columns is a physical column, a row a compact one with
  // the physical rows it owns.  With zero fill compact index i of an affine map owns the group [i*step,
  // (i+1)*step), of a list the positions up to the next kept one.
  const bool raw = P.part != nullptr;
  const bool fill = !raw && C.fill;
  const bool classes = P.c_rows_mapped || P.c_cols_mapped;
  const Axis rows = raw ? axis_identity(P.M) : P.c_rows_mapped ? w.am : classes ? axis_identity(P.M) : C.rm;
  const Axis cols = raw ? axis_identity(P.N) : P.c_cols_mapped ? w.bn : classes ? axis_identity(P.N) : C.cn;
  float* const out = raw ? P.part + (long)w.split * P.M * P.N : (float*)C.p;
  const long ld = raw ? P.N : MODE == 1 ? C.plane : C.ld;  // (MODE 1: a row is a channel plane)
  const float alpha = raw ? 1.0f : C.alpha, beta = raw ? 0.0f : C.beta;
  const float* const src = raw ? nullptr : (const float*)C.relu_src;
  const bool relu = !raw && C.relu;
  // 16 x 16 tiles whose results own few positions: an element per thread, stored with the zeros that it owns.  Such a
  // product is over in a few thousand clocks, of a wavefront or two per SIMD at 7 - 8 clocks an instruction: every
  // instruction counts (64 x 784 -> 1024, dp = 2: the tables and the general loop below took 3300 of a workgroup's 11400
  // clocks, this takes 1800; the product 6.4 -> 5.9 us).  Four elements a thread of a 32 x 32 tile are no faster so, and
  // slower where a row's zeros are wide apart (4.6 -> 5.2 us at 128 x 683, every third column).
  if (MODE == 0 && BM * BN <= 256 && !classes && beta == 0.0f && rows.kind == AX_AFFINE && cols.kind == AX_AFFINE && (!fill || rows.step * cols.step <= 4)) {
    const int i_ok = imin(P.M, w.am.n), j_ok = imin(P.N, w.bn.n);
    const int lr = tid / BN, lc = tid % BN, i = w.m0 + lr, j = w.n0 + lc;
    if (i >= P.M || j >= P.N) return;
    float x = alpha * sum(lr, lc);
    if (relu) x = fmaxf(x, 0.0f);
    if (i >= i_ok || j >= j_ok) x = 0.0f;  // (beyond the operand: padding of a compact output)
    const int r = rows.off + i * rows.step, c = cols.off + j * cols.step;
    if (src) x = src[(long)r * ld + c] > 0.0f ? x : 0.0f;
    if (!fill) {
      out[(long)r * ld + c] = x;
      return;
    }
    float* o = out + (long)(i * rows.step) * ld + j * cols.step;
    const int na = i == P.M - 1 ? rows.nphys - i * rows.step : rows.step, nb = j == P.N - 1 ? cols.nphys - j * cols.step : cols.step;
    for (int a = 0; a < na; ++a, o += ld)
      for (int b = 0; b < nb; ++b) o[b] = a == rows.off && b == cols.off ? x : 0.0f;
    return;
  }
  const int m_lim = P.c_rows_mapped ? w.am.n : P.M, n_lim = P.c_cols_mapped ? w.bn.n : P.N;
  const int m1 = imin(w.m0 + BM, m_lim), n1 = imin(w.n0 + BN, n_lim);
  // physical row of every row of the tile, -1 beyond the matrix (a class's last block may end beyond it), and
  // what a row of a list owns with zero fill
  int* const r_p = tab;
  int* const r_lo = tab + BM;
  int* const r_hi = tab + 2 * BM;
  const bool list_fill = fill && rows.kind != AX_AFFINE;
  for (int lr = tid; lr < BM; lr += 256) {
    const int i = w.m0 + lr;
    int p = -1;
    if (i < m1) {
      if (rows.kind == AX_AFFINE) {
        p = rows.off + i * rows.step;
      } else {
        int lo, hi;
        own_range(rows, i, fill, lo, hi, p);
        r_lo[lr] = lo, r_hi[lr] = hi;
        if (p >= rows.nphys) p = -1;
      }
    }
    r_p[lr] = p;
  }
  __syncthreads();
  const bool walk = fill && cols.kind == AX_AFFINE;   // columns walked by physical position
  const int sc = walk ? cols.step : 1;
  const int c_end = walk && n1 == P.N ? cols.nphys : n1 * sc;
  const int nr = m1 - w.m0, i_ok = classes ? nr : imin(nr, w.am.n - w.m0);
  // Large tiles of plain products that leave dropped columns or rows to be zeroed: runs of four physical columns leave as one
  // store (at any dword).  A thread works out once which of its four are kept and then goes down the rows, the wavefronts'
  // partial tiles summed in place before (the loop below sums them again for each position of a strided map).  Weight
  // gradient, 128 x 2048 -> 2048: dp 2 and 2 21.8 -> 17.6 us, dp 4 and 1 17.2 -> 14.9.  Where nothing is dropped nothing is
  // summed twice and the pass that sums in place costs more (30 x 1024 -> 3000: 16.6 us, in runs 18.0); with tile classes,
  // convolutions and tiles that own no wider rows the setting up does (10.2 -> 10.8 us at 24 x 1472 -> 448 in tiles, 136.6 -> 138 us in
  // three products of a convolution).
  // Tiles of 32 x 32 in an instance of their own (IN_RUNS, f32_leaves_in_runs): the code alone, not run, made other products longer
  // (forward products 0.2 of 5.3 us, three products of 64 x 784 -> 1024 18.66 -> 18.85 us).
  constexpr bool RUNS = MODE == 0 && (BM * BN >= 4096 || IN_RUNS);
  const bool runs = IN_RUNS || (RUNS && !classes && beta == 0.0f && walk && (cols.step > 1 || rows.n < rows.nphys));
  if constexpr (RUNS) if (runs) {
    if constexpr (WK > 1) {  // the partial tiles, summed in place
      for (int e = tid; e < BM * BN; e += 256) {
        const int lr = e / BN, lc = e % BN;
        lds[lr * PITCH + lc] = sum(lr, lc);
      }
      __syncthreads();
    }
    const int c_lo = w.n0 * sc, pieces = (c_end - c_lo + 3) >> 2;
    const int pw = pieces > 128 ? 256 : 1 << (32 - __builtin_clz(imax(pieces, 1) * 2 - 1) - 1);  // threads along a row
    const int pr0 = tid / pw, pc0 = tid % pw, rp = 256 / pw;
    for (int pc = pc0; pc < pieces; pc += pw) {
      const int c = c_lo + 4 * pc, nc = imin(4, c_end - c);
      int lc[4];      // its columns in the tile
      uint32_t m[4];  // kept, and within the operand (beyond it: padding of a compact output, zero)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int d = c + t - cols.off, q = d >= 0 ? (int)fdiv((uint32_t)d, P.col_div) : 0;
        const bool ok = t < nc && d >= 0 && q * sc == d && q < P.N && q < w.bn.n;
        lc[t] = ok ? q - w.n0 : 0;
        m[t] = ok ? ~0u : 0u;
        asm("" : "+v"(m[t]));
      }
      auto store = [&](int r, const float (&x)[4]) {
        float* const o = out + (long)r * ld + c;
        if (nc == 4) {
          *reinterpret_cast<F32Run<4>*>(o) = F32Run<4>{{x[0], x[1], x[2], x[3]}};
        } else {
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (t < nc) o[t] = x[t];
        }
      };
      constexpr int U = 4;  // rows at a time: everything read before anything is stored
#pragma unroll 1
      for (int l0 = pr0; l0 < nr; l0 += U * rp) {
        float x[U][4];
        int pr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int lr = imin(l0 + u * rp, nr - 1);
          pr[u] = l0 + u * rp < nr ? r_p[lr] : -1;
#pragma unroll
          for (int t = 0; t < 4; ++t) x[u][t] = lds[lr * PITCH + lc[t]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          uint32_t row_ok = l0 + u * rp < i_ok ? ~0u : 0u;
          asm("" : "+v"(row_ok));
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            x[u][t] = __uint_as_float(__float_as_uint(alpha * x[u][t]) & m[t] & row_ok);
            if (relu) x[u][t] = fmaxf(x[u][t], 0.0f);
          }
        }
        if (src) {
          float g[U][4];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float* q = src + (long)imax(pr[u], 0) * ld + c;
            if (nc == 4) {
              const F32Run<4> v = *reinterpret_cast<const F32Run<4>*>(q);
#pragma unroll
              for (int t = 0; t < 4; ++t) g[u][t] = v.f[t];
            } else {
#pragma unroll
              for (int t = 0; t < 4; ++t) g[u][t] = t < nc ? q[t] : 0.0f;
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t) x[u][t] = g[u][t] > 0.0f ? x[u][t] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (pr[u] >= 0) store(pr[u], x[u]);
      }
      if (!fill || rows.n == rows.nphys) continue;
      const float zeros[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (list_fill) {
        for (int lr = pr0; lr < nr; lr += rp)
          for (int r = r_lo[lr]; r < r_hi[lr]; ++r)
            if (r != r_p[lr]) store(r, zeros);
      } else {
        // row i owns [i*step, (i+1)*step), the last one also the rest
        for (int lr = pr0; lr < nr; lr += rp)
          for (int g = 0; g < rows.step; ++g) {
            const int r = (w.m0 + lr) * rows.step + g;
            if (g != rows.off && r < rows.nphys) store(r, zeros);
          }
        if (m1 == P.M)
          for (int r = P.M * rows.step + pr0; r < rows.nphys; r += rp) store(r, zeros);
      }
    }
    return;
  }
  for (int c = w.n0 * sc + tc; c < c_end; c += CL) {
    int j = c, clo, chi, cp;
    if constexpr (MODE == 1) {
      const int n = (int)fdiv((uint32_t)j, P.cv.per_img);  // column = (image, position)
      cp = n * (int)C.img_stride + (j - n * P.cv.HoWo);
      clo = cp, chi = cp + 1;
    } else if (walk) {
      const int d = c - cols.off;
      j = d >= 0 ? (int)fdiv((uint32_t)d, P.col_div) : 0;
      const bool kept = d >= 0 && j * sc == d && j < P.N;
      clo = c, chi = c + 1, cp = kept ? c : -1;
      j = kept ? j : w.n0;
    } else if (cols.kind == AX_LIST) {
      own_range(cols, j, fill, clo, chi, cp);
    } else {
      cp = cols.kind == AX_AFFINE ? cols.off + j * cols.step : (cols.off + j / cols.bs * cols.step) * cols.bs + j % cols.bs;
      clo = cp, chi = cp + 1;
      if (cp >= cols.nphys) continue;
    }
    const bool j_ok = classes || j < w.bn.n;   // (beyond the operand: padding of a compact output, zero)
    const int lc = j - w.n0;
    for (int q = clo; q < chi; ++q) {
      // Kept rows: U at a time, everything read before anything is stored, selections by masks (left as conditions
      // every read of the LDS stands behind a branch and is waited for by itself).
      constexpr int U = BM / RP < 8 ? BM / RP : 8;
      const int last_ok = q == cp && j_ok ? i_ok : 0;
#pragma unroll 1
      for (int l0 = tr; l0 < BM; l0 += U * RP) {
        float x[U];
        int pr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) pr[u] = r_p[l0 + u * RP];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = sum(l0 + u * RP, lc);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          uint32_t m = l0 + u * RP < last_ok ? ~0u : 0u;
          asm("" : "+v"(m));
          x[u] = __uint_as_float(__float_as_uint(alpha * x[u]) & m);
        }
        if (beta != 0.0f)
          for (int u = 0; u < U; ++u)
            if (pr[u] >= 0) x[u] += beta * out[(long)pr[u] * ld + q];
        if (relu)
#pragma unroll
          for (int u = 0; u < U; ++u) x[u] = fmaxf(x[u], 0.0f);
        if (src) {
          float g[U];
#pragma unroll
          for (int u = 0; u < U; ++u) g[u] = src[(long)imax(pr[u], 0) * ld + q];
#pragma unroll
          for (int u = 0; u < U; ++u) x[u] = g[u] > 0.0f ? x[u] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (pr[u] >= 0) out[(long)pr[u] * ld + q] = x[u];
      }
      if (!fill || rows.n == rows.nphys) continue;
      // Dropped rows: +0.0, or what beta leaves of them (ReLU and its gradient applied as to any other value)
      auto zero = [&](int r) {
        const long idx = (long)r * ld + q;
        float v = 0.0f;
        if (beta != 0.0f) {
          v = beta * out[idx];
          if (relu) v = fmaxf(v, 0.0f);
          if (src) v = src[idx] > 0.0f ? v : 0.0f;
        }
        out[idx] = v;
      };
      if (list_fill) {
        for (int lr = tr; lr < nr; lr += RP)
          for (int r = r_lo[lr]; r < r_hi[lr]; ++r)
            if (r != r_p[lr]) zero(r);
      } else {
        // row i owns [i*step, (i+1)*step), the last one also the rest
        for (int lr = tr; lr < nr; lr += RP)
          for (int g = 0; g < rows.step; ++g) {
            const int r = (w.m0 + lr) * rows.step + g;
            if (g != rows.off && r < rows.nphys) zero(r);
          }
        if (m1 == P.M)
          for (int r = P.M * rows.step + tr; r < rows.nphys; r += RP) zero(r);
      }
    }
  }
}

template <int AK, int BK, int TM, int TN, int WM, int WN, int WK, int D, int MODE, bool IN_RUNS = false>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(const F32Params P) {
  extern __shared__ float f32_lds[];
  f32_body<AK, BK, TM, TN, WM, WN, WK, D, MODE, IN_RUNS>(P, (int)blockIdx.x, f32_lds);
}

}  // namespace ard
