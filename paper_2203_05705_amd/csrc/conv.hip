// Convolution with dropped input feature maps (Sections 5, 6), channel-level reading:
// one sensitivity score per input feature map, the lowest-scoring maps are dropped and
// their activations, weights and gradients are never loaded.
//
// All three passes are implicit GEMMs on the matrix cores:
//   FWD        Y[co, (n,oh,ow)]  = sum_{tap, c kept}  Wp[co, (tap,c)]  * A[n, c, oh*s+kh-p, ow*s+kw-p]
//   BWD_DATA   dA[c kept, (n,y,x)] = sum_{tap, co}    Wq[c, (tap,co)]  * dY[n, co, y-kh+p, x-kw+p]
//   BWD_WEIGHT dW[co, (c kept,tap)] = sum_{(n,oh,ow)} dY[n, co, oh, ow] * A[n, c, oh*s+kh-p, ow*s+kw-p]
// Wp / Wq are compact repacked copies of the kept-channel weights (tiny, built per call).
//
// Two paths.  bf16 with stride 1: the kept maps are copied once into a zero-bordered
// channels-last grid and the products run on the LDS-direct kernel of fast.hpp (second half of
// this file).  Everything else (fp32, strides): the general engine with loaders that compute
// the patch addresses on the fly, im2col never materialised (first half).
#include <stdlib.h>

#include "engine.hpp"
#include "conv_blocks.hpp"
#include "conv_scatter.hpp"
#include "pattern.hpp"

namespace ard {

// ---- sensitivity score and selection -------------------------------------------------------

// part[y * C + c] = sum over workgroup (c, y)'s share of (n, h, w) of floor(min(|a|, 2^15) * 2^24): exact
// integers, so the result does not depend on the order of summation.  Every workgroup writes its own
// partial (no atomics, nothing to clear beforehand); the selection kernel adds the few partials of a map.
constexpr int kScoreParts = 64;  // at most this many workgroups share a feature map
constexpr int kScorePlanes = 4;  // planes a wavefront reads at a time (x 2 pieces per lane = 8 loads in flight)
template <typename T>
__global__ __launch_bounds__(256) void channel_score_kernel(const T* A, int N, int C, int HW, int n_per_block, int vec,
                                                           unsigned long long* part) {
  constexpr int CE = ElemTraits<T>::CE;
  __shared__ unsigned long long wave_acc[4];
  const int c = blockIdx.x;
  const int n_begin = blockIdx.y * n_per_block;
  const int n_end = min(N, n_begin + n_per_block);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // floor(x * 2^24) for x in [0, 2^15] needs 40 bits; a float-to-64-bit conversion per element made this
  // pass ALU-bound.  Split exactly instead: hi = trunc(x * 2^8) < 2^24, lo = trunc(x * 2^24 - hi * 2^16)
  // < 2^16 (both products and the difference are exact in fp32), floor(x * 2^24) = hi * 2^16 + lo.
  // hi and lo are summed in 32 bits and folded into the 64-bit sum every `flush` (at most 128 elements).
  unsigned long long acc = 0;
  uint32_t acc_hi = 0, acc_lo = 0;
  auto add = [&](T v) {
    const float x = fminf(fabsf(ElemTraits<T>::to_f32(v)), 32768.0f);
    const uint32_t hi = (uint32_t)(x * 256.0f);
    const float lo_f = fmaf(-65536.0f, (float)hi, x * 16777216.0f);
    acc_hi += hi;
    acc_lo += (uint32_t)lo_f;
  };
  auto flush = [&]() {
    acc += ((unsigned long long)acc_hi << 16) + acc_lo;
    acc_hi = acc_lo = 0;
  };
  if (vec) {
    // planes are whole numbers of 16-byte pieces.  A wavefront takes kScorePlanes planes at a time and its
    // lanes two pieces of each: 8 loads, all unconditional (clamped index, contribution zeroed afterwards)
    // so that they are in flight together -- a load behind a branch is waited for before the next is issued.
    const int chunks = HW / CE;
    const int planes = n_end - n_begin;
    const T* const a0 = A + ((long)n_begin * C + c) * HW;
    for (int pb = wave * kScorePlanes; pb < planes; pb += 4 * kScorePlanes)
      for (int cb = lane; cb < chunks; cb += 128) {
        uint4 q[kScorePlanes][2];
#pragma unroll
        for (int u = 0; u < kScorePlanes; ++u) {
          const uint4* pl = reinterpret_cast<const uint4*>(a0 + (long)min(pb + u, planes - 1) * C * HW);
#pragma unroll
          for (int v = 0; v < 2; ++v) q[u][v] = pl[min(cb + 64 * v, chunks - 1)];
        }
#pragma unroll
        for (int u = 0; u < kScorePlanes; ++u)
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const bool live = pb + u < planes && cb + 64 * v < chunks;
            const uint4 z = live ? q[u][v] : uint4{0u, 0u, 0u, 0u};
            const T* e = reinterpret_cast<const T*>(&z);
#pragma unroll
            for (int t = 0; t < CE; ++t) add(e[t]);   // (a zero piece adds nothing)
          }
        flush();
      }
  } else {
    for (int n = n_begin; n < n_end; ++n) {
      const T* p = A + ((long)n * C + c) * HW;
      for (int i = threadIdx.x; i < HW; i += 256) {
        add(p[i]);
        flush();
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (lane == 0) wave_acc[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[(long)blockIdx.y * C + c] = wave_acc[0] + wave_acc[1] + wave_acc[2] + wave_acc[3];
}

// Adds the `parts` partial scores of every map (score_out gets the totals), then drops the n_drop maps that
// come first in ascending (score, index) order; writes the mask (1 = kept) and the ascending kept list
// (ballot + mbcnt compaction, one workgroup).  The rank of a map is counted by four threads, a quarter of the
// other maps each.  From 64 maps on they first count over the scores rounded to 32-bit floats (a map is dropped
// if fewer than n_drop are smaller): one comparison a map from 16-byte LDS reads, where 64-bit scores and
// indices take four and more (384 maps 20.6 -> 7.3 us, 389 15.1 -> 7.7, 64 to 127 maps 1.07 times as fast;
// fewer gain nothing).  Only if maps with the same rounded score make that more than n_drop is the whole count
// done again over scores and indices (all scores alike: 1.06 to 1.25 times as long as that count alone).
// IN_LDS: the scores fit the staging array (else they are re-read from memory).
// The code is kept short on purpose: a single workgroup that runs once pays every instruction-cache line it
// touches with a fetch from memory (3 KB of straight-line code took 10 us for 256 maps).
template <bool IN_LDS>
__global__ __launch_bounds__(1024) void channel_select_kernel(const unsigned long long* part, int parts,
                                                             unsigned long long* score_out, int C, int n_drop, uint8_t* mask,
                                                             int* keep, int* count, int pad_keep) {
  constexpr int STAGED = 4096;
  __shared__ unsigned long long staged[IN_LDS ? STAGED : 1];
  __shared__ uint4 rounded[IN_LDS ? STAGED / 4 : 1];
  __shared__ int wave_tot[16];
  __shared__ int running_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t* const round = reinterpret_cast<uint32_t*>(rounded);
  if (tid == 0) running_s = 0;
  for (int i = tid; i < C; i += 1024) {
    unsigned long long t = 0;
#pragma unroll 1
    for (int y0 = 0; y0 < parts; y0 += 8) {
      unsigned long long v[8];  // eight unconditional loads in flight (clamped index, contribution zeroed)
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(long)min(y0 + u, parts - 1) * C + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) t += y0 + u < parts ? v[u] : 0ull;
    }
    score_out[i] = t;
    if (IN_LDS) staged[i] = t, round[i] = __float_as_uint((float)t);
  }
  const int quads = (C + 3) / 4;
  if (IN_LDS && C + tid < 4 * quads) round[C + tid] = ~0u;
  if (!IN_LDS) __threadfence_block();
  __syncthreads();
  const int n_kept = min(max(C - n_drop, 0), C);
  const bool count_all = n_kept > 0 && n_kept < C;
#pragma unroll 1
  for (int exact = IN_LDS && C >= 64 ? 0 : 1; exact < 2; ++exact) {
    for (int base = 0; base < C; base += 256) {
      const int c = base + (tid >> 2), part_id = tid & 3;
      int rank = 0;
      if (c < C && count_all) {
        if (IN_LDS && !exact) {
          const uint32_t s = round[c];
#pragma unroll 4
          for (int q = part_id; q < quads; q += 4) {
            const uint4 o = rounded[q];
            rank += (o.x < s ? 1 : 0) + (o.y < s ? 1 : 0) + (o.z < s ? 1 : 0) + (o.w < s ? 1 : 0);
          }
        } else {
          const unsigned long long s = IN_LDS ? staged[c] : score_out[c];
#pragma unroll 4
          for (int o = part_id; o < C; o += 4) {
            const unsigned long long so = IN_LDS ? staged[o] : score_out[o];
            rank += (so < s || (so == s && o < c)) ? 1 : 0;
          }
        }
      }
      rank += __shfl_xor(rank, 1, 64);
      rank += __shfl_xor(rank, 2, 64);
      const bool kept = c < C && part_id == 0 && n_kept > 0 && (rank >= n_drop || !count_all);
      if (c < C && part_id == 0) mask[c] = kept ? 1 : 0;
      const unsigned long long bal = __ballot(kept);
      const int r = __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0));
      if (lane == 0) wave_tot[wave] = __popcll(bal);
      __syncthreads();
      int before = running_s, total = 0;
#pragma unroll 1
      for (int w = 0; w < 16; ++w) {
        int t = wave_tot[w];
        if (w < wave) before += t;
        total += t;
      }
      if (kept) keep[before + r] = c;
      __syncthreads();
      if (tid == 0) running_s += total;
      __syncthreads();
    }
    if (running_s == n_kept) break;
    __syncthreads();  // (everyone has read the count)
    if (tid == 0) running_s = 0;
    __syncthreads();
  }
  if (tid == 0 && count) *count = n_kept;
  if (pad_keep)  // (the list has room for every channel: what is not kept reads -1)
    for (int i = n_kept + tid; i < C; i += 1024) keep[i] = -1;
}

// ---- weight repacking ------------------------------------------------------------------------

// flip == 0: out[r = co][tap][q = kept c] = Wt[co][keep[q]][tap]            (rows = Cout, inner = Ck)
// flip == 1: out[r = kept c][tap][q = co] = Wt[co][keep[r]][taps-1-tap]    (rows = Ck, inner = Cout)
template <typename T>
__global__ void pack_weights_kernel(const T* Wt, const int* keep, int C, int taps, int rows, int inner, int flip,
                                    T* out) {
  const long total = (long)rows * taps * inner;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int q = (int)(idx % inner);
  const int tap = (int)((idx / inner) % taps);
  const int r = (int)(idx / ((long)inner * taps));
  long src = flip ? ((long)q * C + (keep ? keep[r] : r)) * taps + (taps - 1 - tap) : ((long)r * C + (keep ? keep[q] : q)) * taps + tap;
  out[idx] = Wt[src];
}

// ---- implicit-GEMM operand loaders ---------------------------------------------------------------

struct ConvGeom {
  int N, Cin, Hin, Win;      // tensor the patches are cut from
  int Hout, Wout;            // position grid (one GEMM column per (n, oh, ow))
  int KH, KW, stride, pad_h, pad_w;
  int Ck;                    // gathered channels per tap
  const int* chan;           // channel list (NULL = identity)
  // block-based sensitivity-aware pattern (Section 5.2.2): entry (p, q) of an image's input matrix,
  // q = (channel * KH + kh) * KW + kw, is absent when blk[(n * RB + p / bx) * CB + q / by] == 0
  const uint8_t* blk;
  int bx, by, RB, CB;
};

// B operand of FWD / BWD_DATA: row = position (n, oh, ow), contraction index k = tap*Ck + cc.
template <typename T, int ROWS>
struct PatchLoader {
  static constexpr int CE = ElemTraits<T>::CE;
  static constexpr int PASSES = ROWS / 32;
  static constexpr int NREG = PASSES;
  const T* src;
  ConvGeom g;
  int K;
  long ibase[PASSES];
  int bband[PASSES];  // (n * RB + row band) * CB of this thread's position (block pattern only)
  int ih0[PASSES], iw0[PASSES];
  bool rvalid[PASSES];
  int lr[PASSES], lc[PASSES];

  __device__ __forceinline__ void init(const void* p, const ConvGeom& geom, int row0, int tid) {
    src = (const T*)p;
    g = geom;
    K = g.KH * g.KW * g.Ck;
    const int hw = g.Hout * g.Wout;
    const long ntot = (long)g.N * hw;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      int r, c;
      if (ROWS >= 64) {
        constexpr int RP = ROWS >= 64 ? ROWS / 64 : 1;
        r = (tid & 63) + 64 * (ps % RP);
        c = (tid >> 6) + 4 * (ps / RP);
      } else {
        r = tid & 31;
        c = tid >> 5;
      }
      lr[ps] = r;
      lc[ps] = c;
      const long j = (long)row0 + r;
      rvalid[ps] = j < ntot;
      const int n = rvalid[ps] ? (int)(j / hw) : 0;
      const int rem = rvalid[ps] ? (int)(j - (long)n * hw) : 0;
      const int oh = rem / g.Wout, ow = rem - oh * g.Wout;
      ibase[ps] = (long)n * g.Cin * g.Hin * g.Win;
      ih0[ps] = oh * g.stride - g.pad_h;
      iw0[ps] = ow * g.stride - g.pad_w;
      bband[ps] = g.blk ? (n * g.RB + rem / g.bx) * g.CB : 0;
    }
  }

  __device__ __forceinline__ void load(int k0, uint4 (&regs)[PASSES]) const {
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      const int kc = k0 + lc[ps] * CE;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (rvalid[ps] && kc < K) {
        T tmp[CE];
        int tap = kc / g.Ck, cc = kc - tap * g.Ck;
#pragma unroll
        for (int e = 0; e < CE; ++e) {
          while (cc >= g.Ck) {
            cc -= g.Ck;
            ++tap;
          }
          T x = 0;
          if (kc + e < K) {
            const int kh = tap / g.KW, kw = tap - kh * g.KW;
            const int ih = ih0[ps] + kh, iw = iw0[ps] + kw;
            if (ih >= 0 && ih < g.Hin && iw >= 0 && iw < g.Win) {
              const int ch = g.chan ? g.chan[cc] : cc;
              if (!g.blk || g.blk[bband[ps] + (ch * g.KH * g.KW + tap) / g.by])
                x = src[ibase[ps] + ((long)ch * g.Hin + ih) * g.Win + iw];
            }
          }
          tmp[e] = x;
          ++cc;
        }
        v = *reinterpret_cast<const uint4*>(tmp);
      }
      regs[ps] = v;
    }
  }

  __device__ __forceinline__ void store(uint4* tile, const uint4 (&regs)[PASSES]) const {
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) tile[swz(lr[ps], lc[ps])] = regs[ps];
  }
};

struct ConvGemmParams {
  Operand Wp;       // packed weights [M x K], contraction-contiguous
  const void* src;  // activations (FWD) or output gradient (BWD_DATA)
  ConvGeom g;
  OutMat C;
  int M, K;
  long Ncols;
  int tiles_n;
};

template <typename T, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void conv_gemm_kernel(const ConvGemmParams P) {
  constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
  __shared__ uint4 lds[2 * (BM + BN) * LDS_ROW_U4];
  const int tid = threadIdx.x;
  const int mb = blockIdx.x / P.tiles_n, nb = blockIdx.x % P.tiles_n;
  const int m0 = mb * BM, n0 = nb * BN;
  bool act[TM][TN];
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int im = 0; im < TM; ++im)
#pragma unroll
    for (int in = 0; in < TN; ++in) {
      act[im][in] = true;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[im][in][v] = 0.0f;
    }
  if (P.K > 0) {
    LoaderKC<T, BM, 256> la;
    PatchLoader<T, BN> lb;
    la.init(P.Wp, axis_identity(P.K), m0, tid);
    lb.init(P.src, P.g, n0, tid);
    gemm_mainloop<T, BM, BN, WGM, WGN>(la, lb, 0, P.K, lds, acc, act);
  }
  gemm_epilogue<T, BM, BN, WGM, WGN>(P.C, acc, m0, n0, P.M, (int)P.Ncols);
}

// Data gradient under the block pattern (Section 5.2.2).  An entry (p, q) of a dropped block of the input
// matrix receives no gradient, so the term of (input channel c, output position p, filter tap) counts or
// not as a whole: whether it does depends on the output row (c), the output column (the input pixel, which
// with the tap fixes p) and the tap, on no operand alone.  The contraction therefore runs tap by tap into
// a second accumulator that is added where the mask keeps the entry.  P.g is the geometry of the ordinary
// data gradient (positions = input pixels, source = dY, taps flipped, stride 1) and carries the mask with
// RB, CB of the forward input matrices; Cin_fwd = P.M channels, all kept.
template <typename T, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void conv_bwd_data_blocks_kernel(const ConvGemmParams P) {
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  __shared__ uint4 lds[2 * (BM + BN) * LDS_ROW_U4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int mb = blockIdx.x / P.tiles_n, nb = blockIdx.x % P.tiles_n;
  const int m0 = mb * BM, n0 = nb * BN;
  const ConvGeom& g = P.g;
  bool act[TM][TN];
  f32x16_t acc[TM][TN], tacc[TM][TN];
#pragma unroll
  for (int im = 0; im < TM; ++im)
#pragma unroll
    for (int in = 0; in < TN; ++in) {
      act[im][in] = true;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[im][in][v] = 0.0f;
    }
  // this lane's output columns: image and input pixel
  int img[TN], ph[TN], pw[TN];
  bool cvalid[TN];
  const int hw = g.Hout * g.Wout;
#pragma unroll
  for (int in = 0; in < TN; ++in) {
    const long j = (long)n0 + wn * WTN + in * 32 + (lane & 31);
    cvalid[in] = j < P.Ncols;
    img[in] = cvalid[in] ? (int)(j / hw) : 0;
    const int rem = cvalid[in] ? (int)(j - (long)img[in] * hw) : 0;
    ph[in] = rem / g.Wout;
    pw[in] = rem - ph[in] * g.Wout;
  }
  LoaderKC<T, BM, 256> la;
  PatchLoader<T, BN> lb;
  la.init(P.Wp, axis_identity(P.K), m0, tid);
  ConvGeom plain = g;
  plain.blk = nullptr;
  lb.init(P.src, plain, n0, tid);
  const int taps = g.KH * g.KW;
  for (int tap = 0; tap < taps; ++tap) {
#pragma unroll
    for (int im = 0; im < TM; ++im)
#pragma unroll
      for (int in = 0; in < TN; ++in)
#pragma unroll
        for (int v = 0; v < 16; ++v) tacc[im][in][v] = 0.0f;
    lb.K = (tap + 1) * g.Ck;  // the patch loader returns zeros beyond this tap's output channels
    gemm_mainloop<T, BM, BN, WGM, WGN>(la, lb, tap * g.Ck, (tap + 1) * g.Ck, lds, tacc, act);
    const int fh = tap / g.KW, fw = tap - fh * g.KW;        // flipped tap the loader walked
    const int kh = g.KH - 1 - fh, kw = g.KW - 1 - fw;        // the filter tap it stands for
#pragma unroll
    for (int in = 0; in < TN; ++in) {
      const int oh = ph[in] - g.pad_h + fh, ow = pw[in] - g.pad_w + fw;   // output position of this term
      if (!cvalid[in] || oh < 0 || oh >= g.Hin || ow < 0 || ow >= g.Win) continue;
      const uint8_t* band = g.blk + (long)(img[in] * g.RB + (oh * g.Win + ow) / g.bx) * g.CB;
#pragma unroll
      for (int im = 0; im < TM; ++im)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int c = m0 + wm * WTM + im * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
          if (c < P.M && band[((c * g.KH + kh) * g.KW + kw) / g.by]) acc[im][in][v] += tacc[im][in][v];
        }
    }
  }
  gemm_epilogue<T, BM, BN, WGM, WGN>(P.C, acc, m0, n0, P.M, (int)P.Ncols);
}

// A operand of BWD_WEIGHT: row = co, contraction index k = (n, oh, ow) over dY[N, Cout, Ho, Wo].
template <typename T, int ROWS>
struct GradRowLoader {
  static constexpr int CE = ElemTraits<T>::CE;
  static constexpr int PASSES = ROWS / 32;
  static constexpr int NREG = PASSES;
  const T* src;
  int Cout, HW, vec;
  long K;
  int row[PASSES];
  bool rvalid[PASSES];
  int lr[PASSES], lc;

  __device__ __forceinline__ void init(const void* p, int cout, int hw, long k, int v, int row0, int tid) {
    src = (const T*)p;
    Cout = cout;
    HW = hw;
    K = k;
    vec = v;
    lc = tid & 7;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      lr[ps] = (tid >> 3) + 32 * ps;
      row[ps] = row0 + lr[ps];
      rvalid[ps] = row[ps] < Cout;
    }
  }
  __device__ __forceinline__ void load(int k0, uint4 (&regs)[PASSES]) const {
    const long kc = (long)k0 + lc * CE;
    const int n = (int)(kc / HW);
    const int p = (int)(kc - (long)n * HW);
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (rvalid[ps] && kc < K) {
        const T* base = src + ((long)n * Cout + row[ps]) * HW;
        if (vec && p + CE <= HW) {
          v = *reinterpret_cast<const uint4*>(base + p);
        } else {
          T tmp[CE];
          int nn = 0, pp = p;
#pragma unroll
          for (int e = 0; e < CE; ++e) {
            if (pp >= HW) {
              pp -= HW;
              ++nn;
            }
            tmp[e] = (kc + e < K) ? base[(long)nn * Cout * HW + pp] : (T)0;
            ++pp;
          }
          v = *reinterpret_cast<const uint4*>(tmp);
        }
      }
      regs[ps] = v;
    }
  }
  __device__ __forceinline__ void store(uint4* tile, const uint4 (&regs)[PASSES]) const {
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) tile[swz(lr[ps], lc)] = regs[ps];
  }
};

// B operand of BWD_WEIGHT: row j = (kept channel, tap), contraction index k = (n, oh, ow).
template <typename T, int ROWS>
struct PatchColLoader {
  static constexpr int CE = ElemTraits<T>::CE;
  static constexpr int PASSES = ROWS / 32;
  static constexpr int NREG = PASSES;
  const T* src;
  ConvGeom g;
  long K;
  long rbase[PASSES];
  int kh[PASSES], kw[PASSES];
  int cblk[PASSES];  // column block of this row's (channel, tap) (block pattern only)
  bool rvalid[PASSES];
  int lr[PASSES], lc;

  __device__ __forceinline__ void init(const void* p, const ConvGeom& geom, int row0, int tid) {
    src = (const T*)p;
    g = geom;
    const int taps = g.KH * g.KW;
    K = (long)g.N * g.Hout * g.Wout;
    lc = tid & 7;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      lr[ps] = (tid >> 3) + 32 * ps;
      const int j = row0 + lr[ps];
      rvalid[ps] = j < g.Ck * taps;
      const int cc = rvalid[ps] ? j / taps : 0;
      const int tap = rvalid[ps] ? j - cc * taps : 0;
      const int ch = g.chan ? g.chan[cc] : cc;
      rbase[ps] = (long)ch * g.Hin * g.Win;
      kh[ps] = tap / g.KW;
      kw[ps] = tap - kh[ps] * g.KW;
      cblk[ps] = g.blk ? (ch * taps + tap) / g.by : 0;
    }
  }
  __device__ __forceinline__ void load(int k0, uint4 (&regs)[PASSES]) const {
    const long kc = (long)k0 + lc * CE;
    const int hw = g.Hout * g.Wout;
    const int n0 = (int)(kc / hw);
    const int p0 = (int)(kc - (long)n0 * hw);
    const int oh0 = p0 / g.Wout, ow0 = p0 - oh0 * g.Wout;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (rvalid[ps] && kc < K) {
        T tmp[CE];
        int n = n0, oh = oh0, ow = ow0;
#pragma unroll
        for (int e = 0; e < CE; ++e) {
          if (ow >= g.Wout) {
            ow = 0;
            if (++oh >= g.Hout) {
              oh = 0;
              ++n;
            }
          }
          T x = 0;
          if (kc + e < K) {
            const int ih = oh * g.stride - g.pad_h + kh[ps], iw = ow * g.stride - g.pad_w + kw[ps];
            if (ih >= 0 && ih < g.Hin && iw >= 0 && iw < g.Win &&
                (!g.blk || g.blk[(n * g.RB + (oh * g.Wout + ow) / g.bx) * g.CB + cblk[ps]]))
              x = src[(long)n * g.Cin * g.Hin * g.Win + rbase[ps] + (long)ih * g.Win + iw];
          }
          tmp[e] = x;
          ++ow;
        }
        v = *reinterpret_cast<const uint4*>(tmp);
      }
      regs[ps] = v;
    }
  }
  __device__ __forceinline__ void store(uint4* tile, const uint4 (&regs)[PASSES]) const {
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) tile[swz(lr[ps], lc)] = regs[ps];
  }
};

struct ConvWgradParams {
  const void* dY;
  const void* A;
  ConvGeom g;
  float* part;   // [splits][Cout][Nn] fp32 partial sums
  int Cout, Nn, dy_vec;
  long K;
  int k_per_split;
  int tiles_n;
};

template <typename T, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void conv_wgrad_kernel(const ConvWgradParams P) {
  constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
  __shared__ uint4 lds[2 * (BM + BN) * LDS_ROW_U4];
  const int tid = threadIdx.x;
  const int mb = blockIdx.x / P.tiles_n, nb = blockIdx.x % P.tiles_n;
  const int m0 = mb * BM, n0 = nb * BN;
  const int split = blockIdx.y;
  const long kb = (long)split * P.k_per_split;
  const long ke = kb + P.k_per_split < P.K ? kb + P.k_per_split : P.K;
  bool act[TM][TN];
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int im = 0; im < TM; ++im)
#pragma unroll
    for (int in = 0; in < TN; ++in) {
      act[im][in] = true;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[im][in][v] = 0.0f;
    }
  if (kb < ke) {
    GradRowLoader<T, BM> la;
    PatchColLoader<T, BN> lb;
    la.init(P.dY, P.Cout, P.g.Hout * P.g.Wout, P.K, P.dy_vec, m0, tid);
    lb.init(P.A, P.g, n0, tid);
    gemm_mainloop<T, BM, BN, WGM, WGN>(la, lb, (int)kb, (int)ke, lds, acc, act);
  }
  OutMat C{};
  C.p = P.part + (long)split * P.Cout * P.Nn;
  C.ld = P.Nn;
  C.rm = axis_identity(P.Cout);
  C.cn = axis_identity(P.Nn);
  C.out_f32 = 1;
  C.alpha = 1.0f;
  gemm_epilogue<T, BM, BN, WGM, WGN>(C, acc, m0, n0, P.Cout, P.Nn);
}

// dWt[co][c][tap] = rank[c] >= 0 ? sum over splits of part[s][co][rank[c]*taps + tap] : 0
template <typename T>
__global__ void conv_wgrad_reduce_kernel(const float* part, const int* rank, int splits, int Cout, int C, int taps,
                                         int Nn, int kept_only, T* dWt) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long total = (long)Cout * C * taps;
  if (idx >= total) return;
  const int tap = (int)(idx % taps);
  const int c = (int)((idx / taps) % C);
  const int co = (int)(idx / ((long)taps * C));
  float s = 0.0f;
  const int r = rank[c];
  if (r < 0 && kept_only) return;
  if (r >= 0)
    for (int sp = 0; sp < splits; ++sp) s += part[((long)sp * Cout + co) * Nn + (long)r * taps + tap];
  dWt[idx] = ElemTraits<T>::from_f32(s);
}

__global__ void rank_from_keep_kernel(const int* keep, int n_keep, int C, int* rank) {
  for (int c = threadIdx.x; c < C; c += blockDim.x) rank[c] = -1;
  __syncthreads();
  for (int j = threadIdx.x; j < n_keep; j += blockDim.x) rank[keep[j]] = j;
}


// ---- bf16, stride 1: channels-last grid + LDS-direct implicit GEMM ----------------------------------
//
// The kept feature maps are copied once into a zero-bordered channels-last grid
// T[(n*Hg + h + oh)*Wg + w + ow][Cp] (compaction of the kept maps and layout change in one pass;
// Cp = kept channels rounded up to 64, extra channels zero).  On that grid the patch of an
// output pixel is, per filter tap, one contiguous Cp-run at a pixel offset that depends on the
// tap only, so the im2col operand streams through 16-byte LDS-direct loads like a plain matrix.

__host__ __device__ static inline int pad64(int n) { return (n + 63) & ~63; }

// Optional mask of the copy (gradients under a block pattern, Section 5.2.2): source pixel p of image n is
// copied iff blk[(n * RB + p / x) * CB + cb] != 0, else it becomes zeros.  blk == NULL: everything is copied.
struct BandMask {
  const uint8_t* blk;
  int RB, CB, cb, x;
};
__device__ __forceinline__ bool band_kept(const BandMask& m, int n, int p) {
  return !m.blk || m.blk[((long)n * m.RB + p / m.x) * m.CB + m.cb] != 0;
}

// position of channel c in the ascending kept list, or -1 (uniform per workgroup where c is)
__device__ __forceinline__ int kept_rank(const int* keep, int n_keep, int c) {
  int lo = 0, hi = n_keep - 1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1, v = keep[mid];
    if (v == c) return mid;
    if (v < c) lo = mid + 1;
    else hi = mid - 1;
  }
  return -1;
}

// planes of dropped channels of an NCHW tensor to +0.0 (the GEMM writes the kept ones); a workgroup
// takes one channel of ZP_IMGS images, 16-byte stores where the planes allow them
constexpr int ZP_IMGS = 8;
struct ZeroPlanesJob {
  uint16_t* dst;
  const int* keep;
  int n_keep, N, C, HW, vec;
  int blocks;  // C * ceil(N / ZP_IMGS) workgroups of 256 threads (0: no job)
};
__device__ __forceinline__ void zero_dropped_planes_body(const ZeroPlanesJob& z, int block) {
  const int c = block % z.C;
  if (kept_rank(z.keep, z.n_keep, c) >= 0) return;
  const int n0 = (block / z.C) * ZP_IMGS, n1 = min(n0 + ZP_IMGS, z.N);
  if (z.vec) {
    const int chunks = z.HW >> 3;
    for (int i = threadIdx.x; i < (n1 - n0) * chunks; i += 256) {
      const int n = n0 + i / chunks, q = i % chunks;
      *reinterpret_cast<uint4*>(z.dst + ((long)n * z.C + c) * z.HW + q * 8) = make_uint4(0, 0, 0, 0);
    }
  } else {
    for (int i = threadIdx.x; i < (n1 - n0) * z.HW; i += 256) z.dst[((long)(n0 + i / z.HW) * z.C + c) * z.HW + i % z.HW] = 0;
  }
}
__global__ __launch_bounds__(256) void zero_dropped_planes_kernel(ZeroPlanesJob z) { zero_dropped_planes_body(z, (int)blockIdx.x); }

// output positions of dropped rows of the input matrix to +0.0 (row-based sensitivity-aware pattern,
// Section 5.2.1: the results of the kept rows fill the same rows of the output, the others are zero);
// one workgroup per (channel, image) plane, eight positions per thread and step
constexpr int ZPX = 8;  // planes (channels of one image) per workgroup
struct ZeroPixelsJob {
  uint16_t* Y;
  const uint8_t* row_mask;
  int Cout, HW;
  int blocks;  // N * ceil(Cout / ZPX) workgroups of 256 threads (0: no job)
  int all;     // 1: zero every position (a plain stream of 16-byte stores; the product that follows writes the kept ones)
};
__device__ __forceinline__ void zero_dropped_pixels_body(const ZeroPixelsJob& z, int block) {
  const int cgs = (z.Cout + ZPX - 1) / ZPX;
  const int co0 = (block % cgs) * ZPX, n = block / cgs;
  const int nco = min(ZPX, z.Cout - co0);
  uint16_t* p = z.Y + ((long)n * z.Cout + co0) * z.HW;
  const uint8_t* m = z.row_mask + (long)n * z.HW;
  const bool vec = (z.HW % 8) == 0 && (((uintptr_t)z.Y | (uintptr_t)z.row_mask) & 15) == 0;
  if (z.all) {  // (host: only with HW % 8 == 0 and Y on a 16-byte boundary)
    uint4* dst = reinterpret_cast<uint4*>(p);
    for (int i = threadIdx.x; i < nco * (z.HW >> 3); i += 256) dst[i] = make_uint4(0, 0, 0, 0);
  } else if (vec) {
    const int chunks = z.HW >> 3;
    for (int i = threadIdx.x; i < nco * chunks; i += 256) {
      const int c = i / chunks, q = (i - c * chunks) * 8;
      const uint2 mk = *reinterpret_cast<const uint2*>(m + q);
      uint16_t* dst = p + (long)c * z.HW + q;
      if ((mk.x | mk.y) == 0) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(0, 0, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (!(((e < 4 ? mk.x : mk.y) >> ((e & 3) * 8)) & 0xff)) dst[e] = 0;
      }
    }
  } else {
    for (int i = threadIdx.x; i < nco * z.HW; i += 256)
      if (!m[i % z.HW]) p[i] = 0;
  }
}

__global__ __launch_bounds__(256) void zero_dropped_pixels_grid_kernel(ZeroPixelsJob z) { zero_dropped_pixels_body(z, (int)blockIdx.x); }

// Block-based pattern on the LDS-direct path (Section 5.2.2).  When a block of the input matrix spans
// whole 64-channel groups over all filter taps (y a multiple of 64 * taps), a kept block is a set of whole
// 64-deep contraction steps of the grid's (tap, channel) order, and a row band of x output positions can be
// laid out as column tiles of its own (padded with entries that store nothing): every tile then contracts
// over the kept blocks of ONE band, and dropped blocks are neither loaded nor multiplied.
// Tile T = ((image * RB + band) * tpb + part) holds positions band*x + part*BN ... of its image.
struct BlockPlan {
  int N, HoWo, x, RB, CB, tpb, BN, taps, CG, cg_per_blk, KB;
};
// kept 64-channel groups of tile T's band (0 for a tile that holds no position)
__device__ __forceinline__ int block_tile_groups(const uint8_t* blk, const BlockPlan& p, int T) {
  const int part = T % p.tpb, band = (T / p.tpb) % p.RB, n = T / (p.tpb * p.RB);
  if (part * p.BN >= p.x || band * p.x + part * p.BN >= p.HoWo) return 0;
  const uint8_t* row = blk + (long)(n * p.RB + band) * p.CB;
  int g = 0;
  for (int cg = 0; cg < p.CG; ++cg) g += row[cg / p.cg_per_blk] ? 1 : 0;
  return g;
}

// One workgroup (256 threads) lays out tile T: its padded pixel list, the list of its kept contraction steps
// and their number.  Where the tile goes in the launch: longest contraction first on every XCD (workgroups
// start in order, so the long ones do not end up alone at the end).  Every workgroup finds the rank of its own
// tile by counting the tiles that come before it (more kept groups, or as many and a lower index): no pass of
// its own, no hand-over.  order = 0: tile T stays at T.
constexpr int kBlockOrderMaxTiles = 1 << 11;  // (each of n workgroups reads n keys)
struct BlockPlanJob {
  const uint8_t* blk;
  BlockPlan p;
  int tiles, order;
  int *pix, *kb_list, *kb_cnt;
  int blocks;  // = tiles (0: no job)
};
__device__ __forceinline__ void block_plan_body(const BlockPlanJob& j, int T, int* red4) {
  const BlockPlan& p = j.p;
  const int tid = threadIdx.x;
  int at = T;
  if (j.order) {
    const int mine = block_tile_groups(j.blk, p, T);
    int before = 0;
    for (int U = tid; U < j.tiles; U += 256) {
      const int k = block_tile_groups(j.blk, p, U);
      before += (k > mine || (k == mine && U < T)) ? 1 : 0;
    }
    for (int o = 32; o > 0; o >>= 1) before += __shfl_down(before, o, 64);
    if ((tid & 63) == 0) red4[tid >> 6] = before;
    __syncthreads();
    const int r = red4[0] + red4[1] + red4[2] + red4[3];
    // The kernel deals its work items to the 8 XCDs in contiguous shares [x*n/8, (x+1)*n/8) and a share's
    // workgroups start in order: rank r goes to XCD r % 8, place r / 8 of its share; the last n % 8 ranks
    // fill the shares that are one longer than the others.
    const int even = j.tiles / 8;
    int x = r & 7;
    at = r >> 3;
    if (r >= 8 * even) {
      int q = r - 8 * even;
      at = even;
      for (x = 0; x < 8; ++x) {
        const int size = (int)((long)(x + 1) * j.tiles / 8) - (int)((long)x * j.tiles / 8);
        if (size > even && q-- == 0) break;
      }
    }
    at += (int)((long)x * j.tiles / 8);
  }
  const int part = T % p.tpb, band = (T / p.tpb) % p.RB, n = T / (p.tpb * p.RB);
  for (int i = tid; i < p.BN; i += 256) {
    const int in_band = part * p.BN + i, pos = band * p.x + in_band;
    j.pix[(long)at * p.BN + i] = (in_band < p.x && pos < p.HoWo) ? n * p.HoWo + pos : -1;
  }
  if (tid == 0) {
    int cnt = 0;
    const bool any = part * p.BN < p.x && band * p.x + part * p.BN < p.HoWo;
    const uint8_t* row = j.blk + (long)(n * p.RB + band) * p.CB;
    if (any)
      for (int cg = 0; cg < p.CG; ++cg)  // (all taps of a channel group in a row: they share their lines in L2)
        if (row[cg / p.cg_per_blk])
          for (int tap = 0; tap < p.taps; ++tap) j.kb_list[(long)at * p.KB + cnt++] = tap * p.CG + cg;
    j.kb_cnt[at] = cnt;
  }
}
__global__ __launch_bounds__(256) void block_plan_kernel(BlockPlanJob j) {
  __shared__ int red4[4];
  block_plan_body(j, (int)blockIdx.x, red4);
}

// Ascending list, per column block cb, of the output positions (n * HoWo + p) whose band the pattern keeps, and
// their number (row-based pattern: CB = 1, bands of one position).  Workgroup (cb, g) takes the g-th share of the
// bands; where its part of the list starts is the number of kept positions before the share, which it counts
// itself: no pass of its own, no hand-over.
struct PosListJob {
  const uint8_t* blk;
  int bands, RB, CB, x, HoWo, parts, stride;  // bands = N * RB
  int *list, *cnt;
  int blocks;  // = CB * parts (0: no job)
};
__device__ __forceinline__ int band_positions(const PosListJob& j, int cb, int b) {  // kept positions of band b
  return j.blk[(long)b * j.CB + cb] ? min(j.x, j.HoWo - b % j.RB * j.x) : 0;
}
__device__ __forceinline__ void pos_list_body(const PosListJob& j, int block, int* lds /* [520] */) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cb = block / j.parts, g = block - cb * j.parts;
  const int b0 = (int)((long)g * j.bands / j.parts), b1 = (int)((long)(g + 1) * j.bands / j.parts);
  int before = 0;
  if (j.x == 1 && j.CB == 1 && ((uintptr_t)j.blk & 15) == 0) {
    // bytes of a mask, 16 at a time
    for (int b = tid * 16; b + 16 <= b0; b += 4096) {
      const uint4 v = *reinterpret_cast<const uint4*>(j.blk + b);
      for (uint32_t w : {v.x, v.y, v.z, v.w}) before += __popc((w | ((w & 0x7f7f7f7fu) + 0x7f7f7f7fu)) & 0x80808080u);
    }
    for (int b = (b0 & ~15) + tid; b < b0; b += 256) before += j.blk[b] ? 1 : 0;
  } else {
    for (int b = tid; b < b0; b += 256) before += band_positions(j, cb, b);
  }
  for (int o = 32; o > 0; o >>= 1) before += __shfl_down(before, o, 64);
  if (lane == 0) lds[512 + wave] = before;
  __syncthreads();
  int at = lds[512] + lds[513] + lds[514] + lds[515];
  int* const out = j.list + (long)cb * j.stride;
  for (int c = b0; c < b1; c += 256) {
    const int b = c + tid, len = b < b1 ? band_positions(j, cb, b) : 0;
    int incl = len;
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      incl += lane >= o ? v : 0;
    }
    if (lane == 63) lds[516 + wave] = incl;
    __syncthreads();
    int first = at;
    for (int w = 0; w < 4; ++w) {
      first += w < wave ? lds[516 + w] : 0;
      at += lds[516 + w];
    }
    first += incl - len;
    if (j.x == 1) {
      if (len) out[first] = b / j.RB * j.HoWo + b % j.RB;
    } else {
      // a wavefront takes every fourth band, 64 positions at a time
      lds[tid] = len, lds[256 + tid] = first;
      __syncthreads();
      for (int i = wave; i < min(256, b1 - c); i += 4) {
        const int n = lds[i], to = lds[256 + i], bi = c + i, p0 = bi / j.RB * j.HoWo + bi % j.RB * j.x;
        for (int e = lane; e < n; e += 64) out[to + e] = p0 + e;
      }
    }
    __syncthreads();
  }
  if (g == j.parts - 1 && tid == 0) j.cnt[cb] = at;
}

// Wp[row][tap*Cp + q]: forward (flip = 0): row = output channel, q = kept input channel;
// data gradient (flip = 1): row = kept input channel, q = output channel, taps reversed.
struct PackJob {
  const void* Wt;
  const int* keep;
  int C, taps, rows, inner, Cp, flip;
  void* out;
  int blocks;  // workgroups of 256 threads that cover rows * taps * Cp entries (0: no job)
};
template <typename T> __device__ __forceinline__ void pack_weights_body(const PackJob& j, long idx) {
  const T* const Wt = reinterpret_cast<const T*>(j.Wt);
  const long total = (long)j.rows * j.taps * j.Cp;
  if (idx >= total) return;
  int q, tap, r;
  if (total < (1L << 31)) {  // (32-bit divisions: a fraction of the instructions of 64-bit ones)
    const uint32_t i32 = (uint32_t)idx, a = i32 / (uint32_t)j.Cp;
    q = (int)(i32 - a * (uint32_t)j.Cp);
    r = (int)(a / (uint32_t)j.taps);
    tap = (int)(a - (uint32_t)r * (uint32_t)j.taps);
  } else {
    q = (int)(idx % j.Cp);
    tap = (int)((idx / j.Cp) % j.taps);
    r = (int)(idx / ((long)j.Cp * j.taps));
  }
  T v = (T)0;
  if (q < j.inner)
    v = j.flip ? Wt[((long)q * j.C + (j.keep ? j.keep[r] : r)) * j.taps + (j.taps - 1 - tap)]
               : Wt[((long)r * j.C + (j.keep ? j.keep[q] : q)) * j.taps + tap];
  reinterpret_cast<T*>(j.out)[idx] = v;
}
__global__ void pack_weights_grid_kernel(PackJob j) { pack_weights_body<uint16_t>(j, (long)blockIdx.x * blockDim.x + threadIdx.x); }
static PackJob pack_job(const void* Wt, const int* keep, int C, int taps, int rows, int inner, int Cp, int flip, void* out) {
  return PackJob{Wt, keep, C, taps, rows, inner, Cp, flip, out, (int)(((long)rows * taps * Cp + 255) / 256)};
}

// 8 neighbouring pixels of one channel plane, of which the first `valid` exist: one 16-byte load where the
// address allows it, two 8-byte loads or element by element elsewhere (planes of 14 x 14 or 7 x 7 positions
// do not start on 16-byte boundaries)
__device__ __forceinline__ uint4 load_pixels8(const uint16_t* p, int valid) {
  if (valid >= 8 && (((uintptr_t)p) & 15) == 0) return *reinterpret_cast<const uint4*>(p);
  if (valid >= 8 && (((uintptr_t)p) & 7) == 0) {
    const uint2 a = *reinterpret_cast<const uint2*>(p), b = *reinterpret_cast<const uint2*>(p + 4);
    return make_uint4(a.x, a.y, b.x, b.y);
  }
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (e < valid) w[e >> 1] |= (uint32_t)p[e] << ((e & 1) * 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// The copy, driven from the source side:
// a workgroup reads 64 channels x 64 source pixels with 16-byte loads (a thread takes 8 pixels of two
// neighbouring channels), pairs the channels in registers, transposes the pairs through LDS and writes each
// pixel's 64 channels as 128 contiguous bytes.  The border pixels of an image are dealt to the image's
// workgroups and the margin behind the last image to all of them: every pixel of the grid is written once.
// LDS holds [pixel row][32 channel pairs] without padding: pixel 8q + e sits in row 8e + q and its 16-byte
// groups are exchanged by q's upper bits, which spreads both the 4-byte stores of a wave and its 16-byte
// loads over all banks.
// TILES: the positions that count also leave as GradTiles, and packed weights of conv_scatter.hpp ride along.
template <bool TILES>
__global__ __launch_bounds__(256) void to_grid_src_kernel(const uint16_t* src, const int* chan, int n_chan, int Cs, int Hs,
                                                          int Ws, FastDiv div_ws, int Hg, int Wg, int oh, int ow, int Cp,
                                                          int N,
                                                          long n_pix_total, BandMask bm, uint16_t* dst, PackJob pj,
                                                          ZeroPlanesJob zj, ZeroPixelsJob zp, BlockPlanJob bj, PosListJob lj, ScatterPackJob sj, GradTiles gt, int main_x) {
  __shared__ uint32_t tile[64 * 32];
  __shared__ int red4[4];
  // (workgroups beyond the copy's own pack the weights of the product that follows and zero the planes it will
  // not write: independent small jobs that would otherwise be launches of their own)
  // (they come first in the launch: started last they would be a tail of their own behind the copy)
  const int extra_x = (int)gridDim.x - main_x;
  if ((int)blockIdx.x < extra_x) {
    int b = (int)blockIdx.x * (int)gridDim.y + (int)blockIdx.y;
    if (b < lj.blocks) return pos_list_body(lj, b, reinterpret_cast<int*>(tile));
    b -= lj.blocks;
    if constexpr (TILES) {
      if (b < sj.blocks) return scatter_pack_body(sj, b);
      b -= sj.blocks;
    }
    if (b < pj.blocks) pack_weights_body<uint16_t>(pj, (long)b * 256 + threadIdx.x);
    else if (b < pj.blocks + zj.blocks) zero_dropped_planes_body(zj, b - pj.blocks);
    else if (b < pj.blocks + zj.blocks + zp.blocks) zero_dropped_pixels_body(zp, b - pj.blocks - zj.blocks);
    else if (b < pj.blocks + zj.blocks + zp.blocks + bj.blocks) block_plan_body(bj, b - pj.blocks - zj.blocks - zp.blocks, red4);
    return;
  }
  const int HW = Hs * Ws;
  const int px_tiles = (HW + 63) / 64;
  // Channel rows start at any multiple of 2 * HW bytes, so a tile's 128-byte runs straddle cache lines that the
  // neighbouring pixel tile reads too.  Workgroups are dealt to the 8 XCDs in turn: XCD x takes the x-th eighth
  // of the tiles in order, so the second read of a line finds it in that XCD's L2 (half the fetched bytes).
  const int even = main_x / 8, bx = (int)blockIdx.x - extra_x;
  const int m = bx < 8 * even ? (bx & 7) * even + (bx >> 3) : bx;
  const int n = m / px_tiles, tile_j = m - n * px_tiles, p0 = tile_j * 64;
  const int c0 = blockIdx.y * 64;
  const int t = threadIdx.x;
  const int cp = t >> 3, q = t & 7;  // channel pair, piece of 8 pixels
  uint4 v0 = make_uint4(0, 0, 0, 0), v1 = v0;
  {
    const int c = c0 + 2 * cp, p = p0 + q * 8;
    if (p < HW) {
      if (c < n_chan) v0 = load_pixels8(src + ((long)n * Cs + (chan ? chan[c] : c)) * HW + p, HW - p);
      if (c + 1 < n_chan) v1 = load_pixels8(src + ((long)n * Cs + (chan ? chan[c + 1] : c + 1)) * HW + p, HW - p);
    }
  }
  // masked copy: which of the tile's 64 pixels count is the same for all of its channels, looked up once
  __shared__ uint8_t piece_keep[8];
  if (bm.blk) {
    if (t < 8) {
      unsigned bits = 0;
      for (int e = 0; e < 8; ++e) {
        const int p = p0 + t * 8 + e;
        if (p < HW && band_kept(bm, n, p)) bits |= 1u << e;
      }
      piece_keep[t] = (uint8_t)bits;
    }
    __syncthreads();
  }
  // tiles of the kept positions: which ones, and (cols) how many of the image lie before this workgroup's
  __shared__ uint64_t tile_keep;
  if constexpr (TILES) {
    if (t < 64) {
      const int p = p0 + t, band = (p < HW ? p : HW - 1) / gt.x;
      bool k = false;
      for (int cb = 0; cb < gt.CB; ++cb) k |= grad_kept(gt, n, band, cb);
      const uint64_t bits = __ballot(k && p < HW);
      if (t == 0) tile_keep = bits;
    }
    if (gt.cols) {
      int before = 0;
      const uint8_t* const m = gt.mask + (long)n * HW;
      for (int p = t; p < p0; p += 256) before += m[p] ? 1 : 0;
      for (int o = 32; o > 0; o >>= 1) before += __shfl_down(before, o, 64);
      if ((t & 63) == 0) red4[t >> 6] = before;
    }
  }
  {
    uint32_t lo[4] = {v0.x, v0.y, v0.z, v0.w}, hi[4] = {v1.x, v1.y, v1.z, v1.w};
    if (bm.blk) {
      const unsigned bits = piece_keep[q];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (!((bits >> e) & 1)) {
          lo[e >> 1] &= (e & 1) ? 0x0000ffffu : 0xffff0000u;
          hi[e >> 1] &= (e & 1) ? 0x0000ffffu : 0xffff0000u;
        }
    }
    const int col = (((cp >> 2) ^ (q & 6)) << 2) | (cp & 3);
#pragma unroll
    for (int e = 0; e < 8; ++e)  // pixel e of the piece: channel c in the low half, c + 1 in the high half
      tile[(e * 8 + q) * 32 + col] = __builtin_amdgcn_perm(hi[e >> 1], lo[e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
  }
  __syncthreads();
  const uint64_t keep = TILES ? tile_keep : 0;
  int rank0 = p0;
  if (TILES && gt.cols) {
    rank0 = red4[0] + red4[1] + red4[2] + red4[3];
    if (blockIdx.y == 0 && t < 64 && p0 + t < HW) {
      const int p = p0 + t, rank = rank0 + __builtin_popcountll(keep & ((1ull << t) - 1)), row = (int)fdiv((uint32_t)p, div_ws);
      if (keep >> t & 1) gt.cols[(long)n * gt.TI * 16 + rank] = (uint16_t)p;
      if (row * Ws == p) gt.row_start[(long)n * (Hs + 1) + row] = rank;
      if (p == HW - 1) gt.row_start[(long)n * (Hs + 1) + Hs] = rank + (int)(keep >> t & 1);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (t >> 3) + 32 * i, c8 = t & 7;  // LDS row, group of 8 channels
    const int q = r & 7, at = 8 * q + (r >> 3), p = p0 + at;
    if (p >= HW) continue;
    if (TILES && (keep >> at & 1)) {
      const int rank = gt.cols ? rank0 + __builtin_popcountll(keep & ((1ull << at) - 1)) : p;
      const long step = ((long)n * gt.TI + (rank >> 4)) * (Cp / 32) + c0 / 32 + (c8 >> 2);
      reinterpret_cast<uint4*>(gt.tiles)[step * 64 + (c8 & 3) * 16 + (rank & 15)] = *reinterpret_cast<const uint4*>(&tile[r * 32 + ((c8 ^ (q & 6)) << 2)]);
    }
    const int h = (int)fdiv((uint32_t)p, div_ws), w = p - h * Ws;
    const long g = ((long)n * Hg + h + oh) * Wg + w + ow;
    *reinterpret_cast<uint4*>(dst + g * Cp + c0 + c8 * 8) = *reinterpret_cast<const uint4*>(&tile[r * 32 + ((c8 ^ (q & 6)) << 2)]);
  }
  // zero pass, for this workgroup's 64 channels.  The border of image n: `top` whole rows above, `bot` below,
  // then per image row ow pixels on the left and the rest of `side` on the right; border index b of the image
  // belongs to workgroup b * px_tiles / B of the image's px_tiles.
  const uint4 zero = make_uint4(0, 0, 0, 0);
  const int top = oh * Wg, bot = (Hg - oh - Hs) * Wg, side = Wg - Ws, B = top + bot + Hs * side;
  const int b0 = (int)((long)tile_j * B / px_tiles), b1 = (int)((long)(tile_j + 1) * B / px_tiles);
  for (int b = b0 + (t >> 3); b < b1; b += 32) {
    int pos;
    if (b < top) pos = b;
    else if (b < top + bot) pos = (oh + Hs) * Wg + (b - top);
    else {
      const int s = b - top - bot, row = s / (side > 0 ? side : 1), k = s - row * side;
      pos = (oh + row) * Wg + (k < ow ? k : k + Ws);
    }
    *reinterpret_cast<uint4*>(dst + ((long)n * Hg * Wg + pos) * Cp + c0 + (t & 7) * 8) = zero;
  }
  // the margin behind the last image, 32 pixels per workgroup
  for (long g = (long)N * Hg * Wg + (long)bx * 32 + (t >> 3); g < n_pix_total; g += (long)main_x * 32)
    *reinterpret_cast<uint4*>(dst + g * Cp + c0 + (t & 7) * 8) = zero;
}

// ---- fp32, stride 1: zero-bordered channel planes + the fp32 matrix kernels ---------------------------
//
// The kept feature maps are copied once into planes with a zero border, [N][Cp][plane] (Cp a multiple of 16, plane a
// multiple of 16, both filled up with zeros): a tap is then a constant offset into a plane, no load needs a bounds
// test, and the products of fast32.hpp read the planes as they are (forward and data gradient: channels of a tap
// along the contraction, pixels along a plane; weight gradient: pixels of a plane along the contraction).  The
// general engine computed every element's patch address and tested it against the border.  N=64, C=Cout=64, 32x32,
// 3x3, half of the channels kept (2.4 GFLOP a pass): forward 136 -> 32 us, data gradient 193 -> 29, weight gradient
// 165 -> 33, copies 6.5 + 8.8 + 12.9 us.
struct PlaneCopy {
  const float* src;
  const int* chan;   // kept channels (NULL: all)
  int n_chan, Cs, Hs, Ws, oh, ow, Wg, Cp, plane, N;
  FastDiv by_plane4, by_cp, by_wg;  // plane / 4, Cp, Wg
  long total4;       // 16-byte pieces of the planes and the margin behind them
  BandMask bm;
  float* dst;
  int blocks;        // workgroups of 256 threads (0: no job)
};
__device__ __forceinline__ void plane_copy_body(const PlaneCopy& p, int block) {
  const long e = (long)block * 256 + threadIdx.x;
  if (e >= p.total4) return;
  const uint32_t pc = fdiv((uint32_t)e, p.by_plane4);  // (image, channel)
  const int q0 = (int)((uint32_t)e - pc * (uint32_t)(p.plane >> 2)) * 4;
  const int n = (int)fdiv(pc, p.by_cp), c = (int)pc - n * p.Cp;
  const bool live = n < p.N && c < p.n_chan;
  const float* s = p.src + ((long)(live ? n : 0) * p.Cs + (live ? (p.chan ? p.chan[c] : c) : 0)) * p.Hs * p.Ws;
  int h = (int)fdiv((uint32_t)q0, p.by_wg), w = q0 - h * p.Wg;
  h -= p.oh, w -= p.ow;
  float v[4];
  bool ok[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    ok[t] = live && (unsigned)h < (unsigned)p.Hs && (unsigned)w < (unsigned)p.Ws;
    if (ok[t] && p.bm.blk) ok[t] = band_kept(p.bm, n, h * p.Ws + w);
    v[t] = s[ok[t] ? h * p.Ws + w : 0];  // (unconditional loads, four in flight)
    if (++w == p.Wg - p.ow) w = -p.ow, ++h;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = ok[t] ? v[t] : 0.0f;
  *reinterpret_cast<float4*>(p.dst + e * 4) = make_float4(v[0], v[1], v[2], v[3]);
}
// up to two copies, the packed weights and the zeros of dropped planes: one launch, the small jobs first
__global__ __launch_bounds__(256) void to_planes_kernel(PackJob pj, ZeroPlanesJob zj, PlaneCopy a, PlaneCopy b) {
  int x = (int)blockIdx.x;
  if (x < pj.blocks) return pack_weights_body<float>(pj, (long)x * 256 + threadIdx.x);
  x -= pj.blocks;
  if (x < zj.blocks) return zero_dropped_planes_body(zj, x);
  x -= zj.blocks;
  if (x < a.blocks) return plane_copy_body(a, x);
  plane_copy_body(b, x - a.blocks);
}
static PlaneCopy plane_copy(const void* src, const int* chan, int n_chan, int Cs, int Hs, int Ws, int N, int oh, int ow, int Wg, int plane,
                            long margin, float* dst, BandMask bm) {
  PlaneCopy p{};
  p.src = (const float*)src, p.chan = chan, p.n_chan = n_chan, p.Cs = Cs, p.Hs = Hs, p.Ws = Ws, p.oh = oh, p.ow = ow, p.Wg = Wg;
  p.Cp = (n_chan + 15) & ~15, p.plane = plane, p.N = N, p.bm = bm, p.dst = dst;
  p.by_plane4 = fast_div((uint32_t)(plane >> 2)), p.by_cp = fast_div((uint32_t)p.Cp), p.by_wg = fast_div((uint32_t)Wg);
  p.total4 = ((long)N * p.Cp * plane + margin) / 4;
  p.blocks = (int)((p.total4 + 255) / 256);
  return p;
}

// output positions of dropped rows of the input matrix to +0.0 (row-based sensitivity-aware pattern,
// Section 5.2.1: the results of the kept rows fill the same rows of the output, the others are zero);
// one workgroup per (channel, image) plane
template <typename T>
__global__ __launch_bounds__(256) void zero_dropped_pixels_kernel(T* Y, const uint8_t* row_mask, int Cout, int HW) {
  const int co = blockIdx.x, n = blockIdx.y;
  T* p = Y + ((long)n * Cout + co) * HW;
  const uint8_t* m = row_mask + (long)n * HW;
  for (int i = threadIdx.x; i < HW; i += 256)
    if (!m[i]) p[i] = (T)0;
}

// out = Y with the positions of dropped rows of the input matrix as +0.0 (the gradient of a row pattern's
// forward pass only arrives on kept positions); one workgroup per (channel, image) plane
template <typename T>
__global__ __launch_bounds__(256) void mask_pixels_kernel(const T* Y, const uint8_t* row_mask, int Cout, int HW, T* out) {
  const int co = blockIdx.x, n = blockIdx.y;
  const long base = ((long)n * Cout + co) * HW;
  const uint8_t* m = row_mask + (long)n * HW;
  for (int i = threadIdx.x; i < HW; i += 256) out[base + i] = m[i] ? Y[base + i] : (T)0;
}
// the same with the mask of one column block of a block pattern: position p of image n is kept iff
// blk[(n * RB + p / x) * CB + cb] != 0
template <typename T>
__global__ __launch_bounds__(256) void mask_bands_kernel(const T* Y, const uint8_t* blk, int RB, int CB, int cb, int x, int Cout,
                                                         int HW, T* out) {
  const int co = blockIdx.x, n = blockIdx.y;
  const long base = ((long)n * Cout + co) * HW;
  const uint8_t* m = blk + (long)n * RB * CB + cb;
  for (int i = threadIdx.x; i < HW; i += 256) out[base + i] = m[(long)(i / x) * CB] ? Y[base + i] : (T)0;
}
// the forward pass of a column block adds what its kept bands give: out = (first ? 0 : out) + (kept ? Y : 0)
__global__ __launch_bounds__(256) void add_bands_kernel(const float* Y, const uint8_t* blk, int RB, int CB, int cb, int x, FastDiv by_x, int Cout,
                                                        int HW, float* out) {
  const int co = blockIdx.x, n = blockIdx.y;
  const long base = ((long)n * Cout + co) * HW;
  const uint8_t* m = blk + (long)n * RB * CB + cb;
  for (int i = threadIdx.x; i < HW; i += 256) {
    const float y = m[(long)fdiv((uint32_t)i, by_x) * CB] ? Y[base + i] : 0.0f;
    out[base + i] = cb ? out[base + i] + y : y;
  }
}
__global__ void iota_kernel(int* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = i;
}

// dW[co][c][tap] = sum over splits of part[sp][co][tap*Cp + rank(c)] (dropped channels: +0.0).
// A thread owns one kept synapse (co, tap, r): consecutive threads read consecutive r (coalesced), the
// loads of the splits are independent and summed in split order.  The same launch writes the zeros of
// the dropped channels (its first gridDim.x - zero_blocks workgroups sum, the rest zero).
// (column blocks of a pattern: channels lie in groups of `group`, part[sp][co][(r / group) * taps * Cp + tap*Cp +
// r % group] with Cp channels reserved per group; one group else.  keep NULL: every channel.)
template <typename T>
__global__ __launch_bounds__(256) void wgrad_grid_reduce_kernel(const float* part, const int* keep, int n_keep, int splits,
                                                                int Cout, int C, int taps, int Cp, int sum_blocks, int group, int pitch, T* dWt) {
  const int Nn = pitch;
  if ((int)blockIdx.x < sum_blocks) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)Cout * taps * n_keep) return;
    // (the host refuses 2^31 kept synapses or more: 32-bit divisions, a fraction of the instructions of 64-bit ones)
    const uint32_t i32 = (uint32_t)idx, q1 = i32 / (uint32_t)n_keep;
    const int r = (int)(i32 - q1 * (uint32_t)n_keep);
    const int co = (int)(q1 / (uint32_t)taps), tap = (int)(q1 - (uint32_t)co * (uint32_t)taps);
    const int cb = r / group;
    const float* p = part + (long)co * Nn + (cb * taps + tap) * Cp + r - cb * group;
    const long stride = (long)Cout * Nn;
    float s = 0.0f;
    int sp = 0;
    for (; sp + 4 <= splits; sp += 4) {
      const float v0 = p[(sp + 0) * stride], v1 = p[(sp + 1) * stride], v2 = p[(sp + 2) * stride], v3 = p[(sp + 3) * stride];
      s += v0;
      s += v1;
      s += v2;
      s += v3;
    }
    for (; sp < splits; ++sp) s += p[sp * stride];
    dWt[((long)co * C + (keep ? keep[r] : r)) * taps + tap] = ElemTraits<T>::from_f32(s);
    return;
  }
  // zeros of the dropped channels: one thread per (co, c)
  const long idx = (long)(blockIdx.x - sum_blocks) * 256 + threadIdx.x;
  if (idx >= (long)Cout * C) return;
  const int c = (int)(idx % C);
  if (kept_rank(keep, n_keep, c) >= 0) return;
  T* o = dWt + idx * taps;
  for (int t = 0; t < taps; ++t) o[t] = (T)0;
}

struct ConvArgs {
  int32_t mode, dtype, N, C, H, W, Cout, kh, kw, stride, pad, n_keep, Ho, Wo, es;
  int32_t reuse;  // ARD_CONV_REUSE_* bits of the mode argument
  // block-based pattern of the forward pass (ard_conv_fwd_blocks): x-by-y blocks of the input matrices
  const uint8_t* blk;
  int32_t bx, by;
  int32_t kept_only;  // gradients: write the kept channels' part of the output only (the caller covers the rest)
  BandMask dy_mask;   // gradients on the channels-last grids: positions of dY that count (blk == NULL: all)
  // weight gradient on the channels-last grids: contract over the kept positions only (blk == NULL: over all), for each
  // group of `cpb` channels over its own (0: one group)
  PosListJob lists;
  int32_t cpb;
  // data gradient on the channels-last grids: computed over the kept positions only (blk == NULL: over all); `cb` is not
  // used, column block b holds the channels [b * scatter_cpb, (b + 1) * scatter_cpb)
  BandMask scatter;
  int32_t scatter_cpb;
  int32_t pad_keep;  // SELECT: ARD_CONV_PAD_KEEP
};

struct ConvWs {
  unsigned long long* score;
  unsigned long long* score_part;  // [kScoreParts x C] partial scores of the workgroups
  int* rank;
  int* all_chan;   // 0 .. C-1: the kept list of the passes that drop no channel
  char* dy_rows;   // [N, Cout, Ho, Wo] dtype: dY with the dropped rows of a row pattern zeroed
  char* wp;
  float* part;
  uint16_t *grid_a, *grid_y;  // channels-last grids of the fast path (NULL when it does not apply)
  uint16_t* gwp;              // its packed weights
  float* gpart;               // its weight-gradient partial sums
  float *plane_a, *plane_y;   // zero-bordered channel planes of the fp32 path (NULL when it does not apply)
  float *plane_wp, *plane_part;  // its packed weights and weight-gradient partial sums
  size_t plane_part_bytes;
  int *blk_pix, *blk_kb, *blk_cnt;  // block pattern on the fast path: padded pixel list, per-tile block lists and counts
  size_t blk_ints;                  // ints reserved for blk_pix and for blk_kb
  int *pos_list, *pos_cnt;          // kept output positions of every column block of a pattern (pos_blocks at most)
  int pos_blocks;
  uint16_t* tile_cols;  // with dy_rows: GradTiles of the data gradient over the kept positions
  int* tile_rows;
  size_t total;
  int splits;
  int gsplits;  // contraction splits of the fast weight-gradient product
};

// The LDS-direct path: bf16, stride 1, padding no larger than the filter allows for the data
// gradient, and grids small enough for 32-bit element offsets.
static bool conv_fast_ok(const ConvArgs& a);
static int pad16(int n) { return (n + 15) & ~15; }
// Planes of the fp32 path: A with a border of `pad`, dY with the border the data gradient convolves.  For a
// size-preserving filter both have the same rows, and the weight gradient reads dY's bordered plane from its first
// output position on; else it needs dY at the top left of a plane laid out like A's.
struct ConvPlanes {
  int wa, wy, plane_a, plane_y;
  bool same;
  long margin;
};
static ConvPlanes conv_planes(const ConvArgs& a) {
  ConvPlanes g;
  const int ho = a.H + 2 * a.pad - a.kh + 1, wo = a.W + 2 * a.pad - a.kw + 1;
  g.wa = a.W + 2 * a.pad, g.wy = wo + 2 * (a.kw - 1 - a.pad);
  g.plane_a = pad16((a.H + 2 * a.pad) * g.wa), g.plane_y = pad16((ho + 2 * (a.kh - 1 - a.pad)) * g.wy);
  if (g.plane_y < g.plane_a) g.plane_y = g.plane_a;  // (room for the weight gradient's layout as well)
  g.same = a.kh - 1 == 2 * a.pad && a.kw - 1 == 2 * a.pad;
  g.margin = pad16(a.kh * (g.wa > g.wy ? g.wa : g.wy) + a.kw + 16);
  return g;
}
static bool conv_planes_ok(const ConvArgs& a) {
  if (a.dtype != ARD_F32 || a.stride != 1 || a.pad > a.kh - 1 || a.pad > a.kw - 1) return false;
  const ConvPlanes g = conv_planes(a);
  const long lim = 1L << 29;  // elements: 32-bit byte offsets inside a grid and an output
  return (long)a.N * pad16(a.C) * g.plane_a + g.margin < lim && (long)a.N * pad16(a.Cout) * g.plane_y + g.margin < lim &&
         (long)a.N * a.Cout * a.Ho * a.Wo < lim && (long)a.N * a.C * a.H * a.W < lim &&
         (long)(a.Cout > a.C ? a.Cout : a.C) * a.kh * a.kw * pad16(a.Cout > a.C ? a.Cout : a.C) < lim;
}
static long conv_grid_pixels(const ConvArgs& a, int* hg, int* wg);
static int conv_grid_splits(const ConvArgs& a);

static int wgrad_splits(const ConvArgs& a) {
  long tiles = (long)ceil_div(a.Cout, 128) * ceil_div(a.C * a.kh * a.kw, 128);
  long K = (long)a.N * a.Ho * a.Wo;
  long want = (1024 + tiles - 1) / tiles;
  long maxs = (K + 255) / 256;
  long s = want < maxs ? want : maxs;
  return (int)(s < 1 ? 1 : (s > 64 ? 64 : s));
}

static ConvWs conv_ws_layout(char* base, const ConvArgs& a) {
  ConvWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align_up(bytes ? bytes : 1, 256);
    return p;
  };
  const size_t taps = (size_t)a.kh * a.kw;
  w.splits = wgrad_splits(a);
  w.score = (unsigned long long*)take((size_t)a.C * 8);
  w.score_part = (unsigned long long*)take((size_t)a.C * 8 * kScoreParts);
  w.rank = (int*)take((size_t)a.C * 4);
  w.all_chan = (int*)take((size_t)a.C * 4);
  {
    // (dY masked, or its tiles for the data gradient over the kept positions: one pass takes one of them)
    const size_t masked = (size_t)a.N * a.Cout * a.Ho * a.Wo * a.es, tiles = (size_t)a.N * ceil_div(a.Ho * a.Wo, 16) * 16 * pad64(a.Cout) * 2;
    w.dy_rows = take(conv_fast_ok(a) && tiles > masked ? tiles : masked);
  }
  w.wp = take((size_t)a.Cout * a.C * taps * a.es);
  w.part = (float*)take((size_t)w.splits * a.Cout * a.C * taps * 4);
  w.grid_a = w.grid_y = w.gwp = nullptr;
  w.gpart = nullptr;
  w.blk_pix = w.blk_kb = w.blk_cnt = nullptr;
  w.blk_ints = 0;
  w.pos_list = w.pos_cnt = nullptr;
  w.pos_blocks = 0;
  w.tile_cols = nullptr;
  w.tile_rows = nullptr;
  w.gsplits = 1;
  w.plane_a = w.plane_y = w.plane_wp = w.plane_part = nullptr;
  w.plane_part_bytes = 0;
  if (conv_planes_ok(a)) {
    const ConvPlanes g = conv_planes(a);
    const size_t ca = pad16(a.C), cy = pad16(a.Cout), cols = taps * ca;
    w.plane_a = (float*)take(((size_t)a.N * ca * g.plane_a + g.margin) * 4);
    w.plane_y = (float*)take(((size_t)a.N * cy * g.plane_y + g.margin) * 4);
    w.plane_wp = (float*)take((size_t)(a.Cout > a.C ? a.Cout : a.C) * taps * (ca > cy ? ca : cy) * 4);
    // partial sums of the weight gradient: about a thousand 64 x 64 tiles over all splits
    const long tiles = (long)ceil_div(a.Cout, 64) * ceil_div((int)cols, 64);
    const long s = 1024 / tiles < 1 ? 1 : 1024 / tiles > 256 ? 256 : 1024 / tiles;
    w.plane_part_bytes = (size_t)s * a.Cout * cols * 4;
    w.plane_part = (float*)take(w.plane_part_bytes);
  }
  if (conv_fast_ok(a)) {
    int hg, wg;
    const long pix = conv_grid_pixels(a, &hg, &wg);
    w.gsplits = conv_grid_splits(a);
    const size_t cpa = pad64(a.C), cpy = pad64(a.Cout);
    w.grid_a = (uint16_t*)take((size_t)pix * cpa * 2);
    w.grid_y = (uint16_t*)take((size_t)pix * cpy * 2);
    int ks, passes;
    size_t frag_bytes, rows_bytes = (size_t)(a.Cout > a.C ? a.Cout : a.C) * taps * (cpa > cpy ? cpa : cpy) * 2;
    scatter_passes(a.C, a.Cout, (int)taps, ks, passes, frag_bytes);
    w.gwp = (uint16_t*)take(rows_bytes > frag_bytes ? rows_bytes : frag_bytes);
    w.gpart = (float*)take((size_t)w.gsplits * a.Cout * taps * cpa * 4);
    // tiles padded to at most twice the output positions; at most 128 blocks per tile of at least 128 positions
    w.blk_ints = 2 * (size_t)a.N * a.Ho * a.Wo + 512;
    w.blk_pix = (int*)take(w.blk_ints * 4);
    w.blk_kb = (int*)take(w.blk_ints * 4);
    w.blk_cnt = (int*)take((w.blk_ints / 128 + 1) * 4 * 2);  // counts, then the tiles' places in the launch
    w.pos_blocks = imin(pad64(a.C) / 64, 16);
    w.pos_list = (int*)take((size_t)w.pos_blocks * a.N * a.Ho * a.Wo * 4);
    w.pos_cnt = (int*)take((size_t)w.pos_blocks * 4);
    w.tile_cols = (uint16_t*)take((size_t)a.N * ceil_div(a.Ho * a.Wo, 16) * 16 * 2);
    w.tile_rows = (int*)take((size_t)a.N * (a.Ho + 1) * 4);
  }
  w.total = off;
  return w;
}


static bool conv_fast_ok(const ConvArgs& a) {
  if (a.dtype != ARD_BF16 || a.stride != 1) return false;
  if (a.pad > a.kh - 1 || a.pad > a.kw - 1) return false;
  int hg, wg;
  const long pix = conv_grid_pixels(a, &hg, &wg);
  const long cmax = pad64(a.C > a.Cout ? a.C : a.Cout);
  return pix * cmax < (1L << 31) && (long)a.kh * a.kw * cmax < (1L << 24);
}

// Pixels of the largest grid any mode builds (input grid with its border, or the output grid
// bordered for the data gradient), plus the margin the shifted reads of the weight gradient
// and the 64-pixel tiles of the copy kernel may touch.
static long conv_grid_pixels(const ConvArgs& a, int* hg, int* wg) {
  const int ho = a.H + 2 * a.pad - a.kh + 1, wo = a.W + 2 * a.pad - a.kw + 1;
  const int h1 = a.H + 2 * a.pad, w1 = a.W + 2 * a.pad;
  const int h2 = ho + 2 * (a.kh - 1 - a.pad), w2 = wo + 2 * (a.kw - 1 - a.pad);
  *hg = h1 > h2 ? h1 : h2;
  *wg = w1 > w2 ? w1 : w2;
  const long margin = (long)a.kh * *wg + a.kw + 128;
  return (long)a.N * *hg * *wg + margin;
}

static int conv_grid_splits(const ConvArgs& a) {
  const long tiles = (long)ceil_div(a.Cout, 128) * ceil_div(a.kh * a.kw * pad64(a.C), 128);
  long s = 512 / tiles;  // about two 128 x 128 workgroups per CU
  return (int)(s < 1 ? 1 : (s > 64 ? 64 : s));
}

static bool al16c(const void* p) { return ((uintptr_t)p & 15) == 0; }

static int32_t to_grid(const void* src, const int* chan, int n_chan, int Cs, int Hs, int Ws, int N, int Hg, int Wg, int oh,
                       int ow, int Cp, long margin, uint16_t* dst, hipStream_t stream, BandMask bm = BandMask{},
                       PackJob pj = PackJob{}, ZeroPlanesJob zj = ZeroPlanesJob{}, ZeroPixelsJob zp = ZeroPixelsJob{},
                       BlockPlanJob bj = BlockPlanJob{}, PosListJob lj = PosListJob{}, ScatterPackJob sj = ScatterPackJob{}, GradTiles gt = GradTiles{}) {
  const long total = (long)N * Hg * Wg + margin;
  if (oh < 0 || ow < 0 || Hg < oh + Hs || Wg < ow + Ws) return fail(ARD_EINVAL, "grid copy: the image does not fit the grid");
  const int main_x = N * ceil_div(Hs * Ws, 64);
  const int gy = Cp / 64;
  dim3 grid((unsigned)(main_x + ceil_div(pj.blocks + zj.blocks + zp.blocks + bj.blocks + lj.blocks + sj.blocks, gy)), (unsigned)gy);
  ARD_LAUNCH_NAMED("to_grid_src_kernel", (gt.tiles ? to_grid_src_kernel<true> : to_grid_src_kernel<false>), grid, dim3(256), 0, stream,
                   (const uint16_t*)src, chan, n_chan, Cs, Hs, Ws, fast_div((uint32_t)Ws), Hg, Wg, oh, ow, Cp, N, total, bm, dst, pj, zj, zp, bj, lj,
                   sj, gt, main_x);
  ARD_LAUNCH_CHECK("to_grid_src_kernel");
  return ARD_OK;
}

// The tile of a product of `rows` rows by `npix` pixels on the grids, and its cost (2304 times the rounds it takes, by their cost).
struct GridTile {
  int bm, bn;
  long cost;
};
static GridTile pick_grid_tile(int rows, int npix) {
  // A launch runs in rounds: one workgroup of a large shape fills a CU (256 at a time), three of the 64 x 64 shape share
  // one (768 at a time).  Costs of a round, a 256 x 256 round being 100, from launches of two whole rounds, contractions of
  // 1152 and 2304 (us: 31 and 51 of 64 x 64, 50 and 84 of the smaller large ones, 64 and 107 of 256 x 192, 67 and 111 of
  // 128 x 384, 78 and 131 of 128 x 448, 79 and 134 of 256 x 256); how often the pixels are read, with 128 to 512 rows,
  // makes no difference.  A third of a round's cost goes by the tiles in it: those of a last round that is not full are
  // over sooner (256 rows, 100352 pixels: 392 tiles of 256 x 256 take 74 and 122 us, 448 of 128 x 448, cheaper by the
  // round, 75 and 125).  Lowest cost wins: over 44 layers (8 - 200 images, 7 x 7 - 56 x 56, 64 - 512 channels and rows) the
  // choice is within 0.2 % of the best in the mean, within 4 % at most.  (Costs and layers measured with a core of 32 x 32 x 16 MFMAs;
  // with that of 16 x 16 x 32 the same choice is within 0.35 and 5 %, 82 layers, forward and data gradient.)
  static const struct { int bm, bn, slots, cost; } kTiles[] = {{64, 64, 768, 40}, {128, 256, 256, 63}, {256, 128, 256, 63}, {256, 192, 256, 81},
                                                               {128, 384, 256, 83}, {128, 448, 256, 97}, {256, 256, 256, 100}};
  GridTile best{0, 0, -1};
  for (const auto& t : kTiles) {
    if (t.bm > 64 && rows <= t.bm / 2) continue;
    const long n = (long)ceil_div(rows, t.bm) * ceil_div(npix, t.bn), rounds = (n + t.slots - 1) / t.slots;
    const long c = (2 * rounds * t.slots + n) * (768 / t.slots) * t.cost;
    if (best.cost < 0 || c <= best.cost) best = GridTile{t.bm, t.bn, c};
  }
  return best;
}

// Y[row][pixel] = sum_k Wp[row][k] * im2col[pixel][k] on the grid; NCHW output
// force_bn / kb_*: the block-based pattern's launch (column tile fixed by its plan, per-tile contraction lists)
static int32_t conv_grid_gemm(const uint16_t* Wp, int rows, int K, const uint16_t* grid_t, long grid_pixels,
                              const ConvMap& cv, void* out, hipStream_t stream, int force_bn = 0,
                              const int* kb_list = nullptr, const int* kb_cnt = nullptr, int kb_stride = 0) {
  FastParams F{};
  F.A = Wp;
  F.B = grid_t;
  F.a_elems = (long)rows * K;
  F.b_elems = grid_pixels * cv.Cp;
  F.C = (uint16_t*)out;
  F.lda = K;
  F.ldb = cv.Cp;
  F.am = axis_identity(rows);
  F.bn = axis_identity(cv.npix);
  F.k = axis_identity(K);
  F.alpha = 1.0f;
  F.splits = 1;
  F.M = rows;
  F.N = cv.npix;
  F.cv = cv;
  F.cv.set_divisors(K / cv.Cp);
  F.kb_list = kb_list, F.kb_cnt = kb_cnt, F.kb_stride = kb_stride;
  int bm, bn;
  if (force_bn) {
    bm = force_bn == 128 || rows > 128 ? 256 : 128;
    bn = force_bn;
  } else {
    const GridTile t = pick_grid_tile(rows, cv.npix);
    bm = t.bm, bn = t.bn;
  }
  F.tiles_m = ceil_div(rows, bm);
  F.tiles_n = ceil_div(cv.npix, bn);
  const long tiles = (long)F.tiles_m * F.tiles_n;
  if (tiles >= (1L << 24)) return fail(ARD_ESHAPE, "convolution too large for one launch");
  F.total_tiles = (int)tiles;
  set_bands(F, direct_group_m(F.total_tiles));
  const int grid = direct_plain_grid(F.total_tiles);
  if (bm == 256 && bn == 256) return launch_direct_kernel<true, true, 256, 256, 8, 1>(F, grid, stream);
  if (bm == 256 && bn == 192) return launch_direct_kernel<true, true, 256, 192, 8, 1>(F, grid, stream);
  if (bm == 128 && bn == 384) return launch_direct_kernel<true, true, 128, 384, 8, 1>(F, grid, stream);
  if (bm == 128 && bn == 448) return launch_direct_kernel<true, true, 128, 448, 8, 1>(F, grid, stream);
  if (bm == 256) return launch_direct_kernel<true, true, 256, 128, 8, 1>(F, grid, stream);
  if (bm == 128) return launch_direct_kernel<true, true, 128, 256, 8, 1>(F, grid, stream);
  return launch_direct_kernel<true, true, 64, 64, 4, 1>(F, grid, stream);
}

// Whether the weight gradient can take listed pixels: the kernel multiplies their numbers by 24-bit products (a layer
// beyond contracts over every pixel of dY's masked grid instead).
static bool pos_lists_fit(const ConvArgs& a) { return (long)a.N * (a.H + 2 * a.pad) * (a.W + 2 * a.pad) < (1L << 24); }
// The kept positions of the column blocks of a pattern (bands of x positions, CB blocks), listed in the workspace
static PosListJob pos_list_job(const ConvArgs& a, const uint8_t* blk, int x, int CB, const ConvWs& w) {
  PosListJob j{};
  j.blk = blk, j.HoWo = a.Ho * a.Wo, j.x = x, j.RB = ceil_div(j.HoWo, x), j.CB = CB, j.bands = a.N * j.RB;
  j.parts = imin(imax(j.bands / (x == 1 ? 512 : 32), 1), 128);  // (a share is a few rounds of the workgroup)
  j.stride = a.N * j.HoWo;
  j.list = w.pos_list, j.cnt = w.pos_cnt, j.blocks = CB * j.parts;
  return j;
}

// Whether the forward pass under a block pattern can run over tiles that end anywhere in a band (conv_blocks.hpp).  However
// short the bands and small the layer: against the patch loaders of the general engine, 30 % kept, us, 128 x 256 channels of
// 28 x 28 -> 256 in bands of 1 and 8 positions 7289 and 6900 -> 208 and 198, 8 x 64 of 14 x 14 -> 32 218 -> 14, one image of
// 64 of 7 x 7 -> 16 149 -> 14, two of 512 of 7 x 7 -> 256 1512 -> 49.
static bool block_masked_ok(const ConvArgs& a, const ConvWs& w) {
  const int taps = a.kh * a.kw, CG = pad64(a.C) / 64;
  return w.grid_a && !dev_knobs().no_fast && a.by % (64 * taps) == 0 && CG <= 32 && taps * CG <= 128 && a.kh <= 15 && a.kw <= 15 &&
         (long)ceil_div(a.N * a.Ho * a.Wo, 128) * ceil_div(a.Cout, 64) < (1L << 24);
}

// The column tile (128 or 256 positions) that wastes the least padding, or 0 when this path does not apply.
static int block_fast_tile(const ConvArgs& a, const ConvWs& w) {
  const int taps = a.kh * a.kw;
  if (!w.grid_a || !w.blk_pix || dev_knobs().no_fast || a.Cout <= 64) return 0;
  if (a.by % (64 * taps)) return 0;
  const int CG = pad64(a.C) / 64;
  if (taps * CG > 128) return 0;
  const long hw = (long)a.Ho * a.Wo, RB = ceil_div(a.Ho * a.Wo, a.bx);
  int best = 0;
  long best_len = 0;
  for (int bn : {256, 128}) {
    if (bn == 128 && a.Cout <= 128) continue;  // (the 128-row tile comes with 256 columns only)
    const long len = RB * ceil_div(a.bx, bn) * bn;  // padded positions per image
    if (len > 2 * hw) continue;
    if (!best || len < best_len) best = bn, best_len = len;
  }
  if (!best) return 0;
  const long tiles = (long)a.N * best_len / best;
  // (fewer workgroups than CUs, each a whole CU's: the smaller tiles of conv_blocks.hpp are faster.  Training steps of drawn
  // layers, us, these against those: 44 workgroups 126 and 101, 150 73 and 69, 210 211 and 204, 308 257 and 264, 448 178 and
  // 190, 1344 379 and 426; forward passes of a few: 4 workgroups (288 positions) 19.5 and 13.9, 2 (256) 56 and 28, 1 (256) 11.3
  // and 9.8)
  if (tiles * ceil_div(a.Cout, best == 128 || a.Cout > 128 ? 256 : 128) < 256 && block_masked_ok(a, w)) return 0;
  if ((size_t)(a.N * best_len) > w.blk_ints || (size_t)(tiles * taps * CG) > w.blk_ints || tiles >= (1L << 22)) return 0;
  return best;
}

// (see block_masked_ok)
static int32_t conv_block_fwd(const ConvArgs& a, int Cp, int Hg, int Wg, const ConvWs& w, void* out, hipStream_t stream) {
  BlockFwdParams P{};
  const int taps = a.kh * a.kw;
  P.W = w.gwp, P.grid = w.grid_a, P.Y = (uint16_t*)out, P.blk = a.blk;
  P.ldw = taps * Cp, P.Cp = Cp, P.CG = Cp / 64, P.kh = a.kh, P.kw = a.kw;
  P.HW = a.Ho * a.Wo, P.W_ = a.Wo, P.Cout = a.Cout, P.npix = a.N * P.HW, P.HgWg = Hg * Wg, P.Wg = Wg;
  P.RB = ceil_div(P.HW, a.bx), P.CB = ceil_div(a.C * taps, a.by), P.x = a.bx, P.cg_per_blk = imin(a.by / (64 * taps), 32);
  P.mt = ceil_div(a.Cout, 64), P.total = ceil_div(P.npix, 128) * P.mt;
  P.width = 2;
  for (int m = 16; m > 2 && P.width == 2; m /= 2)
    if (P.HW % (m / 2) == 0 && (uintptr_t)out % m == 0) P.width = m;
  P.by_mt = fast_div((uint32_t)P.mt), P.by_hw = fast_div((uint32_t)P.HW), P.by_w = fast_div((uint32_t)P.W_), P.by_x = fast_div((uint32_t)a.bx);
  // (a lane's last read: the last output position's patch, the last tap of it, inside the grid; rows of W: Cout of them)
  return launch_conv_block_fwd(P, stream);
}

// Whether the data gradient runs over the kept positions (conv_scatter.hpp): planes whose rows fit in LDS, filters that
// keep the image's size, column blocks of whole groups of 16 channels.
static bool scatter_plan(const ConvArgs& a, const ConvWs& w, const BandMask& m, int cpb, ScatterDataParams& P, int& ks) {
  if (!w.grid_a || dev_knobs().no_fast || a.kh - 1 != 2 * a.pad || a.kw - 1 != 2 * a.pad || cpb % 16) return false;
  size_t bytes;
  P = ScatterDataParams{};
  P.taps = a.kh * a.kw;
  scatter_passes(a.C, a.Cout, P.taps, ks, P.passes, bytes);
  P.N = a.N, P.C = a.C, P.H = a.H, P.W_ = a.W, P.HW = a.H * a.W;
  P.kh = a.kh, P.kw = a.kw, P.ph = a.pad, P.pw = a.pad, P.Wl = a.W + a.pad;
  const bool single = m.x == 1 && m.CB == 1;  // (positions one by one: their tiles are made of the kept ones)
  P.t = GradTiles{(uint16_t*)w.dy_rows, single ? w.tile_cols : nullptr, single ? w.tile_rows : nullptr, m.blk, ceil_div(P.HW, 16), m.RB, m.CB, m.x};
  P.steps = pad64(a.Cout) / 32;
  if (P.HW > 65535 || (long)kSdImages * P.t.TI * P.steps * 1024 >= (1L << 32)) return false;  // (positions and offsets of a workgroup)
  P.G = ceil_div(a.C, 16);
  if (!scatter_units(P, ks)) return false;
  const long total = (long)ceil_div(a.N, P.im) * P.bands * P.G;
  if (total >= (1L << 24)) return false;
  P.total = (int)total;
  P.by_groups = fast_div((uint32_t)P.G), P.by_bands = fast_div((uint32_t)P.bands), P.by_hw = fast_div((uint32_t)P.HW);
  P.by_w = fast_div((uint32_t)P.W_), P.by_x = fast_div((uint32_t)m.x), P.by_gpb = fast_div((uint32_t)(cpb / 16));
  return true;
}
// What the kernels for a data gradient take beside what all of them do (launches, the copy of dY), in us, good enough to compare them:
// fitted to 168 drawn row-pattern and 247 block-pattern layers (7 x 7 - 56 x 56, 16 - 512 channels, 3 x 3 and 5 x 5), 30 to 100 %
// kept each, all measured both ways.  Against knowing the faster one, the choice below costs 1 to 3 % in the mean over them up to
// 70 % kept, 6 to 8 % where everything is kept (there nearly half at worst).  The share of kept positions: the 30 % that possibilities of
// 0.3 and 0.7 leave where nothing is sensitive, and some more.  (Both kernels launched, the one to run found by the count on
// the GPU, was 7 % slower with 30 % kept and 12 % faster with all, over the 49 layers whose line lies between: taken back.)
constexpr double kKeptGuess = 0.4;
static double launch_rounds(long n, int slots) { return (2.0 * ((n + slots - 1) / slots) + (double)n / slots) / 3.0; }
// Over the kept positions: a tap of a tile adds its sums in LDS, whatever the channels of dY (5.9: weights double-buffered only).
// Bands of x positions: the fullest workgroups of a round are what it waits for.
static double scatter_us(const ScatterDataParams& P, int ks, double kept, int x) {
  const double rounds = launch_rounds(P.total, P.lds_bytes <= kSdLds ? 512 : 256);
  const double positions = (double)P.im * imin(P.rows >= P.H ? P.H : P.rows + 2 * P.ph, P.H) * P.W_, bands = positions > x ? positions / x : 1.0;
  const double full = kept + std::sqrt(kept * (1.0 - kept) / (bands * rounds)), taps = rounds * P.passes * P.taps;
  return taps * positions * (full < 1.0 ? full : 1.0) / 6400.0 * (ks >= 6 ? 17.2 : 11.3) + taps * ks * 0.0062 + rounds * P.im * P.rows * P.W_ * 0.0042;
}
// Over all positions of a masked copy
static double masked_us(const ConvArgs& a) {
  const int K = a.kh * a.kw * pad64(a.Cout);
  return (3.6 * (K / 64) + 34.6) * 1e-6 * pick_grid_tile(a.C, a.N * a.H * a.W).cost - 3.0;
}
static double block_tiles_us(const ConvArgs& a, const BlockDataParams& P) {
  return launch_rounds((long)a.N * P.tiles_img * P.CB * P.mt, 512) * a.kh * a.kw * P.CG * 0.41 + 2.0;
}
// Data gradient under the block pattern over tiles of positions (conv_blocks.hpp): tiles of 128 positions are whole bands or
// parts of a band, and at least half full (else the passes per column block, whose tiles run over all positions).
static bool block_data_tiles(const ConvArgs& a, const ConvWs& w, BlockDataParams& P) {
  const int taps = a.kh * a.kw, hw = a.H * a.W;
  if (!w.grid_a || dev_knobs().no_fast || a.kh - 1 != 2 * a.pad || a.kw - 1 != 2 * a.pad || a.kh > 15 || a.kw > 15) return false;
  if (a.by % (64 * taps) || (long)a.C * taps % a.by || a.bx % a.W) return false;
  P.RB = ceil_div(hw, a.bx), P.CB = a.C * taps / a.by;
  P.CG = pad64(a.Cout) / 64;
  if (P.RB > 64 || taps * P.CG > 128) return false;
  P.x = a.bx, P.rows_per_band = a.bx / a.W;
  P.bands_per_tile = imax(1, 128 / a.bx), P.parts = ceil_div(a.bx, 128);
  P.tiles_img = P.parts == 1 ? ceil_div(P.RB, P.bands_per_tile) : P.RB * P.parts;
  P.cpb = a.by / taps, P.mt = P.cpb / 64;
  return hw * 2 >= P.tiles_img * 128 && (long)a.N * P.tiles_img * P.CB * P.mt < (1L << 24);
}
static int32_t conv_block_data(const ConvArgs& a, BlockDataParams P, const void* Wt, const void* dYin, void* out, const ConvWs& w,
                               hipStream_t stream) {
  const int taps = a.kh * a.kw, ph = a.kh - 1 - a.pad, pw = a.kw - 1 - a.pad, Cp = pad64(a.Cout), Hg = a.Ho + 2 * ph, Wg = a.Wo + 2 * pw;
  int hgm, wgm;
  (void)conv_grid_pixels(a, &hgm, &wgm);
  const long margin = (long)a.kh * wgm + a.kw + 128;
  // (the kept positions of every group, which the weight gradient of the same workspace contracts over, ride along)
  if (int32_t st = to_grid(dYin, nullptr, a.Cout, a.Cout, a.Ho, a.Wo, a.N, Hg, Wg, ph, pw, Cp, margin, w.grid_y, stream, BandMask{},
                           pack_job(Wt, nullptr, a.C, taps, a.C, a.Cout, Cp, 1, w.gwp), ZeroPlanesJob{}, ZeroPixelsJob{}, BlockPlanJob{}, a.lists))
    return st;
  P.W = w.gwp, P.grid = w.grid_y, P.dA = (uint16_t*)out, P.blk = a.blk;
  P.ldw = taps * Cp, P.Cp = Cp, P.kh = a.kh, P.kw = a.kw, P.ph = ph, P.pw = pw;
  P.H = a.H, P.W_ = a.W, P.C = a.C, P.HgWg = Hg * Wg, P.Wg = Wg;
  P.total = a.N * P.tiles_img * P.CB * P.mt;
  const int hw = a.H * a.W;
  P.width = hw % 8 == 0 && a.bx % 8 == 0 && al16c(out) ? 16 : hw % 2 == 0 && a.bx % 2 == 0 && ((uintptr_t)out & 3) == 0 ? 4 : 2;
  P.by_groups = fast_div((uint32_t)(P.CB * P.mt)), P.by_tiles = fast_div((uint32_t)P.tiles_img), P.by_w = fast_div((uint32_t)a.W);
  // (a lane's last read: the last pixel of the last image through the last tap, inside the grid; rows of W: C of them)
  return launch_conv_block_data(P, stream);
}
static int32_t conv_scatter(ScatterDataParams P, int ks, const ConvWs& w, void* out, hipStream_t stream) {
  P.W = w.gwp, P.dA = (uint16_t*)out;
  const int start = P.bands > 1 ? P.rows * P.W_ : 0;  // (of a band in its plane)
  P.width = 2;
  for (int m = 16; m > 2 && P.width == 2; m /= 2)
    if (P.HW % (m / 2) == 0 && start % (m / 2) == 0 && (uintptr_t)out % m == 0) P.width = m;
  return launch_conv_scatter(ks, P, stream);
}

static int32_t conv_run_grid(const ConvArgs& a, const void* A, const void* Wt, const void* dYin, void* out,
                             const int32_t* d_keep, const uint8_t* row_mask, const ConvWs& w, hipStream_t stream) {
  const int taps = a.kh * a.kw, Ck = a.n_keep;
  int hgm, wgm;
  const long pix_cap = conv_grid_pixels(a, &hgm, &wgm);
  (void)pix_cap;
  // Both grids are laid out the same way whichever pass builds them, so a later pass of the same layer
  // can take the grid an earlier one left in the workspace (ARD_CONV_REUSE_A / ARD_CONV_REUSE_DY):
  // A: zero border of `pad` pixels; dY: zero border of k-1-pad pixels (what the data gradient convolves).
  // The weight gradient wants dY on the grid of A without a border: for a size-preserving filter
  // (k - 1 = 2 pad) that is the bordered dY grid read from (k-1-pad) rows and columns further on.
  const long margin = (long)a.kh * wgm + a.kw + 128;
  const bool same = a.kh - 1 == 2 * a.pad && a.kw - 1 == 2 * a.pad;
  if (a.mode == ARD_CONV_FWD_ROWS) {
    // every channel, only the kept output positions: the product's columns are the listed pixels
    const int Cp = pad64(a.C), Hg = a.H + 2 * a.pad, Wg = a.W + 2 * a.pad, K = taps * Cp;
    // (the zeros of the dropped positions and the packed weights ride in the copy's launch)
    // (with few rows kept, zeros everywhere as one stream cost less than the masked stores of the dropped ones)
    const int fill_all = ((a.Ho * a.Wo) % 8) == 0 && al16c(out) && (long)Ck * 10 <= (long)a.N * a.Ho * a.Wo * 7;
    const ZeroPixelsJob zp{(uint16_t*)out, row_mask, a.Cout, a.Ho * a.Wo, a.N * ceil_div(a.Cout, ZPX), fill_all};
    int32_t st = to_grid(A, nullptr, a.C, a.C, a.H, a.W, a.N, Hg, Wg, a.pad, a.pad, Cp, margin, w.grid_a, stream, BandMask{},
                         pack_job(Wt, nullptr, a.C, taps, a.Cout, a.C, Cp, 0, w.gwp), ZeroPlanesJob{}, zp);
    if (st) return st;
    if (Ck == 0) return ARD_OK;
    ConvMap cv{a.Ho * a.Wo, a.Wo, Hg * Wg, Wg, Cp, a.kw, Ck, a.Cout, nullptr, a.Cout, (const int*)d_keep, a.N * a.Ho * a.Wo, -1};
    return conv_grid_gemm(w.gwp, a.Cout, K, w.grid_a, (long)a.N * Hg * Wg + margin, cv, out, stream);
  }
  if (a.mode == ARD_CONV_FWD) {
    const int Cp = pad64(Ck), Hg = a.H + 2 * a.pad, Wg = a.W + 2 * a.pad, K = taps * Cp;
    int32_t st = ARD_OK;
    const PackJob pj = pack_job(Wt, (const int*)d_keep, a.C, taps, a.Cout, Ck, Cp, 0, w.gwp);
    BlockPlanJob bj{};
    int bn = 0;
    if (a.blk) {
      bn = block_fast_tile(a, w);
      if (!bn && !block_masked_ok(a, w)) return fail(ARD_EUNSUPPORTED, "block pattern outside the fast path");  // (callers test both first)
    }
    if (bn) {
      bj.p = BlockPlan{a.N, a.Ho * a.Wo, a.bx, ceil_div(a.Ho * a.Wo, a.bx), ceil_div(a.C * taps, a.by), ceil_div(a.bx, bn), bn, taps,
                       Cp / 64, a.by / (64 * taps), taps * (Cp / 64)};
      bj.blk = a.blk;
      bj.tiles = bj.blocks = a.N * bj.p.RB * bj.p.tpb;
      bj.order = bj.tiles > 256 && bj.tiles <= kBlockOrderMaxTiles;  // (up to one tile per CU there is nothing to order)
      bj.pix = w.blk_pix, bj.kb_list = w.blk_kb, bj.kb_cnt = w.blk_cnt;
    }
    if (!(a.reuse & ARD_CONV_REUSE_A)) {
      // (the packed weights and the tile plan of a block pattern ride in the copy's launch)
      st = to_grid(A, d_keep, Ck, a.C, a.H, a.W, a.N, Hg, Wg, a.pad, a.pad, Cp, margin, w.grid_a, stream, BandMask{}, pj,
                   ZeroPlanesJob{}, ZeroPixelsJob{}, bj);
    } else {
      ARD_LAUNCH(pack_weights_grid_kernel, dim3((unsigned)pj.blocks), dim3(256), 0, stream, pj);
      ARD_LAUNCH_CHECK("pack_weights_grid_kernel");
      if (bj.blocks) {
        ARD_LAUNCH(block_plan_kernel, dim3((unsigned)bj.blocks), dim3(256), 0, stream, bj);
        ARD_LAUNCH_CHECK("block_plan_kernel");
      }
    }
    if (st) return st;
    if (a.blk && !bn) return conv_block_fwd(a, Cp, Hg, Wg, w, out, stream);
    if (a.blk) {
      const BlockPlan& bp = bj.p;
      const int tiles = bj.tiles;
      // bands of an even number of positions in planes of an even size: the tiles hold whole pairs of neighbours
      const int pairs = (a.bx % 2 == 0) && ((a.Ho * a.Wo) % 2 == 0);
      ConvMap cv{a.Ho * a.Wo, a.Wo, Hg * Wg, Wg, Cp, a.kw, tiles * bn, a.Cout, nullptr, a.Cout, w.blk_pix, a.N * a.Ho * a.Wo, -1, pairs};
      return conv_grid_gemm(w.gwp, a.Cout, K, w.grid_a, (long)a.N * Hg * Wg + margin, cv, out, stream, bn, w.blk_kb, w.blk_cnt,
                            bp.KB);
    }
    ConvMap cv{a.Ho * a.Wo, a.Wo, Hg * Wg, Wg, Cp, a.kw, a.N * a.Ho * a.Wo, a.Cout, nullptr, a.Cout, nullptr, 0, -1};
    return conv_grid_gemm(w.gwp, a.Cout, K, w.grid_a, (long)a.N * Hg * Wg + margin, cv, out, stream);
  }
  if (a.mode == ARD_CONV_BWD_DATA) {
    // dA = dY (bordered by k-1-pad) convolved with the reversed filter, contraction over (tap, co)
    const int ph = a.kh - 1 - a.pad, pw = a.kw - 1 - a.pad;
    const int Cp = pad64(a.Cout), Hg = a.Ho + 2 * ph, Wg = a.Wo + 2 * pw, K = taps * Cp;
    int32_t st = ARD_OK;
    ScatterDataParams sd;
    int ks = 0;
    if (a.scatter.blk && !(a.reuse & ARD_CONV_REUSE_DY) && scatter_plan(a, w, a.scatter, a.scatter_cpb, sd, ks)) {
      const ScatterPackJob sj{(const uint16_t*)Wt, a.C, a.Cout, taps, sd.passes, ks, sd.G, w.gwp, ceil_div(sd.G * sd.passes * taps * ks, 4)};
      // (the kept positions of every group, which the weight gradient of the same workspace contracts over, ride along)
      st = to_grid(dYin, nullptr, a.Cout, a.Cout, a.Ho, a.Wo, a.N, Hg, Wg, ph, pw, Cp, margin, w.grid_y, stream, a.dy_mask, PackJob{},
                   ZeroPlanesJob{}, ZeroPixelsJob{}, BlockPlanJob{}, a.lists, sj, sd.t);
      if (st) return st;
      return conv_scatter(sd, ks, w, out, stream);
    }
    const PackJob pj = pack_job(Wt, (const int*)d_keep, a.C, taps, Ck, a.Cout, Cp, 1, w.gwp);
    ZeroPlanesJob zj{};
    if (Ck < a.C && !a.kept_only) {
      const int hw = a.H * a.W;
      zj = ZeroPlanesJob{(uint16_t*)out, (const int*)d_keep, Ck, a.N, a.C, hw, (int)((hw % 8) == 0 && al16c(out)),
                         a.C * ceil_div(a.N, ZP_IMGS)};
    }
    if (!(a.reuse & ARD_CONV_REUSE_DY)) {
      st = to_grid(dYin, nullptr, a.Cout, a.Cout, a.Ho, a.Wo, a.N, Hg, Wg, ph, pw, Cp, margin, w.grid_y, stream, a.dy_mask, pj, zj,
                   ZeroPixelsJob{}, BlockPlanJob{}, a.lists);
    } else {
      ARD_LAUNCH(pack_weights_grid_kernel, dim3((unsigned)pj.blocks), dim3(256), 0, stream, pj);
      ARD_LAUNCH_CHECK("pack_weights_grid_kernel");
      if (zj.blocks) {
        ARD_LAUNCH(zero_dropped_planes_kernel, dim3((unsigned)zj.blocks), dim3(256), 0, stream, zj);
        ARD_LAUNCH_CHECK("zero_dropped_planes_kernel");
      }
    }
    if (st) return st;
    ConvMap cv{a.H * a.W, a.W, Hg * Wg, Wg, Cp, a.kw, a.N * a.H * a.W, a.C, (const int*)d_keep, Ck, nullptr, 0, -1};
    return conv_grid_gemm(w.gwp, Ck, K, w.grid_y, (long)a.N * Hg * Wg + margin, cv, out, stream);
  }
  // BWD_WEIGHT: contraction over the pixels of the input grid; dY sits on the same grid (top-left
  // aligned, zero elsewhere), the tap shifts the activation grid by (r*Wg + s) pixels.
  const int Cpa = pad64(Ck), Cpy = pad64(a.Cout), Hg = a.H + 2 * a.pad, Wg = a.W + 2 * a.pad;
  int32_t st = ARD_OK;
  if (!(a.reuse & ARD_CONV_REUSE_A))
    st = to_grid(A, d_keep, Ck, a.C, a.H, a.W, a.N, Hg, Wg, a.pad, a.pad, Cpa, margin, w.grid_a, stream);
  if (st) return st;
  // dY: bordered like the data gradient's grid when the filter preserves the size (then shared with it)
  const int ph = same ? a.kh - 1 - a.pad : 0, pw = same ? a.kw - 1 - a.pad : 0;
  const long y_shift = (long)ph * Wg + pw;  // pixels between the bordered grid's origin and dY(., 0, 0)
  // (the lists of kept positions are made in the launch of dY's copy, by either gradient: who shares the copy shares them)
  if (!(a.reuse & ARD_CONV_REUSE_DY))
    st = to_grid(dYin, nullptr, a.Cout, a.Cout, a.Ho, a.Wo, a.N, Hg, Wg, ph, pw, Cpy, margin, w.grid_y, stream, a.dy_mask, PackJob{},
                 ZeroPlanesJob{}, ZeroPixelsJob{}, BlockPlanJob{}, a.lists);
  if (st) return st;
  const bool listed = a.lists.blk != nullptr;
  const int group = a.cpb ? a.cpb : Cpa, groups = a.cpb ? a.lists.CB : 1, cols = taps * group;  // columns of a group of channels
  const int Kq = a.N * Hg * Wg, Nn = groups * cols;
  FastParams F{};
  F.A = w.grid_y + y_shift * Cpy;
  F.B = w.grid_a;
  F.lda = Cpy;
  F.ldb = Cpa;
  F.a_elems = ((long)a.N * Hg * Wg + margin - y_shift) * Cpy;
  F.b_elems = ((long)a.N * Hg * Wg + margin) * Cpa;
  F.am = axis_identity(Cpy);
  F.bn = axis_identity(Nn);
  F.k = axis_identity(Kq);
  F.alpha = 1.0f;
  F.part = w.gpart;
  // tile 256 x 128 (8 wavefronts) when there are enough output channels, else 128 x 128; the
  // contraction is split until every CU has a workgroup (two of the small ones), within the
  // room the workspace has for partial sums
  const bool big = a.Cout > 128;
  const int bm = big ? 256 : 128;
  const long cap = (long)w.gsplits * taps * pad64(a.C) / Nn;
  F.tiles_m = ceil_div(a.Cout, bm);
  F.tiles_n = groups * ceil_div(cols, 128);
  F.total_tiles = F.tiles_m * F.tiles_n;
  int splits = (big ? 256 : 512) / F.total_tiles;
  if (splits > cap) splits = (int)cap;
  const int steps = ceil_div(Kq, 64);
  if (splits > steps) splits = steps;
  if (splits < 1) splits = 1;
  F.splits = splits;
  F.M = a.Cout;
  F.N = Nn;
  F.cv = ConvMap{a.Ho * a.Wo, a.Wo, Hg * Wg, Wg, Cpa, a.kw, 0, 0, nullptr, 0, nullptr, a.N * a.Ho * a.Wo, -1};
  F.cv.set_divisors(taps);
  if (listed) F.li = ListMap{0, a.lists.stride, a.N * a.Ho * a.Wo, ceil_div(cols, 128), cols, a.cpb, group, a.N * Hg * Wg, a.lists.list, a.lists.cnt};
  set_bands(F, direct_group_m(F.total_tiles));
  if (listed)
    st = big ? launch_direct_kernel<false, false, 256, 128, 8, 3>(F, direct_plain_grid(F.total_tiles), stream)
             : launch_direct_kernel<false, false, 128, 128, 4, 3>(F, direct_plain_grid(F.total_tiles), stream);
  else
    st = big ? launch_direct_kernel<false, false, 256, 128, 8, 2>(F, direct_plain_grid(F.total_tiles), stream)
           : launch_direct_kernel<false, false, 128, 128, 4, 2>(F, direct_plain_grid(F.total_tiles), stream);
  if (st) return st;
  if ((long)a.Cout * taps * Ck >= (1L << 31)) return fail(ARD_ESHAPE, "weight gradient beyond 2^31 kept synapses");
  const int sum_blocks = (int)(((long)a.Cout * taps * Ck + 255) / 256);
  const int zero_blocks = Ck < a.C && !a.kept_only ? (int)(((long)a.Cout * a.C + 255) / 256) : 0;
  ARD_LAUNCH(wgrad_grid_reduce_kernel<uint16_t>, dim3((unsigned)(sum_blocks + zero_blocks)), dim3(256), 0, stream, (const float*)w.gpart,
             (const int*)d_keep, Ck, splits, a.Cout, a.C, taps, group, sum_blocks, group, Nn, (uint16_t*)out);
  ARD_LAUNCH_CHECK("wgrad_grid_reduce_kernel");
  return ARD_OK;
}

// The three passes of an fp32 layer on the zero-bordered planes (see to_planes_kernel).
static int32_t conv_run_planes(const ConvArgs& a, const void* A, const void* Wt, const void* dYin, void* out, const int32_t* d_keep,
                               const ConvWs& w, hipStream_t stream) {
  const int taps = a.kh * a.kw, Ck = a.n_keep;
  const ConvPlanes g = conv_planes(a);
  PackJob pj{};
  ZeroPlanesJob zj{};
  PlaneCopy ca{}, cy{};
  auto launch_copies = [&]() -> int32_t {
    ARD_LAUNCH(to_planes_kernel, dim3((unsigned)(pj.blocks + zj.blocks + ca.blocks + cy.blocks)), dim3(256), 0, stream, pj, zj, ca, cy);
    ARD_LAUNCH_CHECK("to_planes_kernel");
    return ARD_OK;
  };
  F32Conv cv{};
  cv.kw = a.kw, cv.taps = taps, cv.by_kw = fast_div((uint32_t)a.kw);
  OutMat C{};
  C.p = out, C.alpha = 1.0f;
  if (a.mode == ARD_CONV_FWD || a.mode == ARD_CONV_BWD_DATA) {
    const bool fwd = a.mode == ARD_CONV_FWD;
    const int rows = fwd ? a.Cout : Ck, inner = fwd ? Ck : a.Cout, Cp = pad16(inner), ho = fwd ? a.Ho : a.H, wo = fwd ? a.Wo : a.W;
    pj = pack_job(Wt, (const int*)d_keep, a.C, taps, rows, inner, Cp, fwd ? 0 : 1, w.plane_wp);
    if (fwd) ca = plane_copy(A, (const int*)d_keep, Ck, a.C, a.H, a.W, a.N, a.pad, a.pad, g.wa, g.plane_a, g.margin, w.plane_a, BandMask{});
    else ca = plane_copy(dYin, nullptr, a.Cout, a.Cout, a.Ho, a.Wo, a.N, a.kh - 1 - a.pad, a.kw - 1 - a.pad, g.wy, g.plane_y, g.margin, w.plane_y, a.dy_mask);
    if (!fwd && Ck < a.C && !a.kept_only)  // (planes of floats as planes of twice as many halves)
      zj = ZeroPlanesJob{(uint16_t*)out, (const int*)d_keep, Ck, a.N, a.C, 2 * a.H * a.W, (int)((a.H * a.W) % 4 == 0 && al16c(out)),
                         a.C * ceil_div(a.N, ZP_IMGS)};
    if (int32_t st = launch_copies()) return st;
    cv.HoWo = ho * wo, cv.Wo = wo, cv.Wg = fwd ? g.wa : g.wy, cv.plane = fwd ? g.plane_a : g.plane_y, cv.Cp = Cp;
    cv.npix = a.N * ho * wo;
    cv.per_row = fast_div((uint32_t)wo), cv.per_img = fast_div((uint32_t)(ho * wo)), cv.steps_inner = fast_div((uint32_t)(Cp / 16));
    C.rm = fwd || !d_keep ? axis_identity(rows) : axis_list(d_keep, rows, a.C);
    C.cn = axis_identity(cv.npix);
    C.plane = ho * wo, C.img_stride = (long)(fwd ? a.Cout : a.C) * ho * wo;
    return f32_conv_product(w.plane_wp, rows, fwd ? w.plane_a : w.plane_y, cv, C, stream);
  }
  // weight gradient: dY on planes laid out like A's
  const int ph = g.same ? a.kh - 1 - a.pad : 0, pw = g.same ? a.kw - 1 - a.pad : 0, Cp = pad16(Ck);
  ca = plane_copy(A, (const int*)d_keep, Ck, a.C, a.H, a.W, a.N, a.pad, a.pad, g.wa, g.plane_a, g.margin, w.plane_a, BandMask{});
  cy = plane_copy(dYin, nullptr, a.Cout, a.Cout, a.Ho, a.Wo, a.N, ph, pw, g.wa, g.plane_a, g.margin, w.plane_y, a.dy_mask);
  if (int32_t st = launch_copies()) return st;
  cv.Wg = g.wa, cv.plane = g.plane_a, cv.Cp = Cp, cv.Co = pad16(a.Cout);
  cv.Wo = a.Wo, cv.npix = a.Ho * g.wa, cv.per_row = fast_div((uint32_t)g.wa);
  cv.by_cp = fast_div((uint32_t)Cp), cv.steps_inner = fast_div((uint32_t)(g.plane_a / 16));
  int splits = 1;
  const int cap = (int)(w.plane_part_bytes / ((size_t)a.Cout * taps * Cp * 4));
  if (int32_t st = f32_conv_wgrad(w.plane_y + (long)ph * g.wa + pw, w.plane_a, cv, a.N, a.Cout, cap, w.plane_part, &splits, stream)) return st;
  if ((long)a.Cout * taps * Ck >= (1L << 31)) return fail(ARD_ESHAPE, "weight gradient beyond 2^31 kept synapses");
  const int sum_blocks = (int)(((long)a.Cout * taps * Ck + 255) / 256);
  const int zero_blocks = Ck < a.C && !a.kept_only ? (int)(((long)a.Cout * a.C + 255) / 256) : 0;
  ARD_LAUNCH(wgrad_grid_reduce_kernel<float>, dim3((unsigned)(sum_blocks + zero_blocks)), dim3(256), 0, stream, (const float*)w.plane_part,
             (const int*)d_keep, Ck, splits, a.Cout, a.C, taps, Cp, sum_blocks, Cp, taps * Cp, (float*)out);
  ARD_LAUNCH_CHECK("wgrad_grid_reduce_kernel");
  return ARD_OK;
}

static int32_t conv_check(ConvArgs& a) {
  if (a.dtype != ARD_F32 && a.dtype != ARD_BF16) return fail(ARD_EDTYPE, "unknown dtype %d", a.dtype);
  if (a.N <= 0 || a.C <= 0 || a.H <= 0 || a.W <= 0 || a.Cout <= 0 || a.kh <= 0 || a.kw <= 0 || a.stride <= 0 || a.pad < 0)
    return fail(ARD_ESHAPE, "non-positive convolution size");
  if (a.H + 2 * a.pad < a.kh || a.W + 2 * a.pad < a.kw) return fail(ARD_ESHAPE, "kernel larger than the padded input");
  a.Ho = (a.H + 2 * a.pad - a.kh) / a.stride + 1;
  a.Wo = (a.W + 2 * a.pad - a.kw) / a.stride + 1;
  a.es = a.dtype == ARD_BF16 ? 2 : 4;
  if ((long)a.N * a.H * a.W > 0x7fffff00L || (long)a.N * a.Ho * a.Wo > 0x7fffff00L || (long)a.C * a.kh * a.kw > 0x7fffff00L)
    return fail(ARD_ESHAPE, "tensor too large for 32-bit position indices");
  return ARD_OK;
}


template <typename T>
static int32_t conv_run(const ConvArgs& a, double rate, const void* A, const void* Wt, const void* dYin, void* out,
                        uint8_t* d_mask, int32_t* d_keep, int32_t* d_count, int64_t* d_score, const ConvWs& w,
                        hipStream_t stream) {
  const int taps = a.kh * a.kw, ce = 16 / a.es;
  if (a.mode == ARD_CONV_SELECT) {
    if (!(rate >= 0.0 && rate <= 1.0)) return fail(ARD_EINVAL, "rate must be in [0,1] (got %g)", rate);
    if (!A || !d_mask || !d_keep) return fail(ARD_EINVAL, "SELECT needs A, d_mask and d_keep");
    if ((long)a.N * a.H * a.W > (1L << 24)) return fail(ARD_ESHAPE, "SELECT needs N*H*W <= 2^24");
    unsigned long long* score = d_score ? (unsigned long long*)d_score : w.score;
    int ysplit = ceil_div(2048, a.C);
    if (ysplit > a.N) ysplit = a.N;
    if (ysplit > kScoreParts) ysplit = kScoreParts;
    if (ysplit < 1) ysplit = 1;
    const int n_per_block = ceil_div(a.N, ysplit);
    const int parts = ceil_div(a.N, n_per_block);
    const int vec = ((a.H * a.W) % ce) == 0 && al16c(A);
    ARD_LAUNCH(channel_score_kernel<T>, dim3(a.C, parts), dim3(256), 0, stream, (const T*)A, a.N, a.C, a.H * a.W,
                       n_per_block, vec, w.score_part);
    ARD_LAUNCH_CHECK("channel_score_kernel");
    const int n_drop = (int)floor(rate * (double)a.C);
    if (a.C <= 4096)
      ARD_LAUNCH(channel_select_kernel<true>, dim3(1), dim3(1024), 0, stream, (const unsigned long long*)w.score_part, parts,
                         score, a.C, n_drop, d_mask, d_keep, d_count, a.pad_keep);
    else
      ARD_LAUNCH(channel_select_kernel<false>, dim3(1), dim3(1024), 0, stream, (const unsigned long long*)w.score_part, parts,
                         score, a.C, n_drop, d_mask, d_keep, d_count, a.pad_keep);
    ARD_LAUNCH_CHECK("channel_select_kernel");
    return ARD_OK;
  }
  if (a.mode == ARD_CONV_FWD_ROWS) {
    // d_keep lists the kept rows (output positions) of the input matrices, n * Ho*Wo + p, ascending;
    // d_mask is the same set as a 0/1 mask
    const long n_rows = (long)a.N * a.Ho * a.Wo;
    if (a.n_keep < 0 || a.n_keep > n_rows) return fail(ARD_EINVAL, "n_keep=%d outside 0..%ld", a.n_keep, n_rows);
    if (!A || !Wt || !out || !d_mask || (a.n_keep > 0 && !d_keep)) return fail(ARD_EINVAL, "FWD_ROWS needs A, Wt, out, d_mask and d_keep");
    if (a.reuse) return fail(ARD_EUNSUPPORTED, "FWD_ROWS builds its own grid");
    if (w.grid_a && !dev_knobs().no_fast) return conv_run_grid(a, A, Wt, nullptr, out, d_keep, d_mask, w, stream);
    // general path (fp32, strides): every position is computed, the dropped ones are zeroed afterwards
    ConvArgs full = a;
    full.mode = ARD_CONV_FWD;
    full.n_keep = a.C;
    int32_t st = conv_run<T>(full, 0.0, A, Wt, nullptr, out, nullptr, nullptr, nullptr, nullptr, w, stream);
    if (st) return st;
    ARD_LAUNCH(zero_dropped_pixels_kernel<T>, dim3(a.Cout, a.N), dim3(256), 0, stream, (T*)out, (const uint8_t*)d_mask, a.Cout,
               a.Ho * a.Wo);
    ARD_LAUNCH_CHECK("zero_dropped_pixels_kernel");
    return ARD_OK;
  }
  if (a.mode == ARD_CONV_BWD_DATA_ROWS || a.mode == ARD_CONV_BWD_WEIGHT_ROWS) {
    // gradients of FWD_ROWS: positions of dropped rows carry no gradient.  dY is copied once with those
    // positions zeroed, then the ordinary passes run over every position with every channel kept.
    if (!dYin || !d_mask || !out) return fail(ARD_EINVAL, "the row-pattern gradients need dYin, d_mask and out");
    // (the reuse flags mean what they mean for the ordinary gradients: the grid of A that FWD_ROWS left, the
    // masked grid of dY that BWD_DATA_ROWS left -- same mask, same layout)
    ConvArgs full = a;
    full.mode = a.mode == ARD_CONV_BWD_DATA_ROWS ? ARD_CONV_BWD_DATA : ARD_CONV_BWD_WEIGHT;
    full.n_keep = a.C;
    const void* dy_use = w.dy_rows;
    int32_t* every = nullptr;  // (no list: every channel)
    if ((w.grid_a || w.plane_a) && !dev_knobs().no_fast) {
      // the pass copies dY into its grid anyway: that copy drops the positions (bands of one row)
      full.dy_mask = BandMask{(const uint8_t*)d_mask, a.Ho * a.Wo, 1, 0, 1};
      dy_use = dYin;
      // The weight gradient runs over the kept positions only, the data gradient where that is expected to be faster and dY has more
      // than 64 channels (30 % kept, us, all positions and the kept ones: 128 x 256 channels of 28 x 28 -> 256 151 and 102, 64 x 512
      // of 14 x 14 -> 512 98 and 56, 112 x 248 of 56 x 56 -> 96 251 and 296; up to 64 channels 0.54 to 1.2 of the speed, in the mean
      // of 51 layers of more than 20 us none; 1 x 1 filters have one tap to gain what writing the tiles costs: 63 x 256 of 56 x 56 -> 80
      // 176 and 192, 78 layers 0.94 to 1.05 of the speed at 30 % kept, in the mean 0.98).  n_keep, where a caller gives it, says how many rows are kept (128 x 256 of 28 x 28 ->
      // 256, all kept: 151 and 211).
      ScatterDataParams sd;
      int ks;
      const long rows = (long)a.N * a.Ho * a.Wo;
      const double kept = a.n_keep > 0 && a.n_keep <= rows ? (double)a.n_keep / (double)rows : kKeptGuess;
      if (a.mode == ARD_CONV_BWD_DATA_ROWS && a.Cout > 64 && a.kh * a.kw > 1 && scatter_plan(a, w, full.dy_mask, pad16(a.C), sd, ks) && scatter_us(sd, ks, kept, 1) <= masked_us(a))
        full.scatter = full.dy_mask, full.scatter_cpb = pad16(a.C);
      if (w.grid_a && pos_lists_fit(a)) full.lists = pos_list_job(a, (const uint8_t*)d_mask, 1, 1, w);
    } else {
      ARD_LAUNCH(iota_kernel, dim3(ceil_div(a.C, 256)), dim3(256), 0, stream, w.all_chan, a.C);
      ARD_LAUNCH_CHECK("iota_kernel");
      every = w.all_chan;
      ARD_LAUNCH(mask_pixels_kernel<T>, dim3(a.Cout, a.N), dim3(256), 0, stream, (const T*)dYin, (const uint8_t*)d_mask, a.Cout,
                 a.Ho * a.Wo, (T*)w.dy_rows);
      ARD_LAUNCH_CHECK("mask_pixels_kernel");
    }
    return conv_run<T>(full, 0.0, A, Wt, dy_use, out, nullptr, every, nullptr, nullptr, w, stream);
  }
  if (a.n_keep < 0 || a.n_keep > a.C) return fail(ARD_EINVAL, "n_keep=%d outside 0..%d", a.n_keep, a.C);
  if (a.n_keep > 0 && a.n_keep < a.C && !d_keep) return fail(ARD_EINVAL, "d_keep is required");
  if (!out) return fail(ARD_EINVAL, "null output pointer");
  const int Ck = a.n_keep;
  if (a.reuse) {
    const bool grid_path = Ck > 0 && w.grid_a;
    if (!grid_path) return fail(ARD_EUNSUPPORTED, "grid reuse needs the bf16 stride-1 path and at least one kept channel");
    if ((a.reuse & ARD_CONV_REUSE_A) && a.mode == ARD_CONV_BWD_DATA) return fail(ARD_EINVAL, "BWD_DATA has no grid of A to reuse");
    if ((a.reuse & ARD_CONV_REUSE_DY) && a.mode == ARD_CONV_FWD) return fail(ARD_EINVAL, "FWD has no grid of dY to reuse");
    if ((a.reuse & ARD_CONV_REUSE_DY) && a.mode == ARD_CONV_BWD_WEIGHT && !(a.kh - 1 == 2 * a.pad && a.kw - 1 == 2 * a.pad))
      return fail(ARD_EUNSUPPORTED, "the weight gradient shares dY's grid with the data gradient only for k - 1 = 2 pad");
    if (dev_knobs().no_fast) {
      // (development switch: every pass runs on the general engine, which builds no grid; nothing to share)
      ConvArgs plain = a;
      plain.reuse = 0;
      return conv_run<T>(plain, rate, A, Wt, dYin, out, d_mask, d_keep, d_count, d_score, w, stream);
    }
  }
  if (Ck > 0 && w.grid_a && a.mode >= ARD_CONV_FWD && a.mode <= ARD_CONV_BWD_WEIGHT && !dev_knobs().no_fast &&
      (!a.blk || (a.mode == ARD_CONV_FWD && (block_fast_tile(a, w) || block_masked_ok(a, w))))) {
    if (a.mode == ARD_CONV_FWD && (!A || !Wt)) return fail(ARD_EINVAL, "FWD needs A and Wt");
    if (a.mode == ARD_CONV_BWD_DATA && (!dYin || !Wt)) return fail(ARD_EINVAL, "BWD_DATA needs dYin and Wt");
    if (a.mode == ARD_CONV_BWD_WEIGHT && (!dYin || !A)) return fail(ARD_EINVAL, "BWD_WEIGHT needs dYin and A");
    return conv_run_grid(a, A, Wt, dYin, out, d_keep, nullptr, w, stream);
  }
  if (Ck > 0 && w.plane_a && !a.blk && !dev_knobs().no_fast) {
    if (a.mode == ARD_CONV_FWD && (!A || !Wt)) return fail(ARD_EINVAL, "FWD needs A and Wt");
    if (a.mode == ARD_CONV_BWD_DATA && (!dYin || !Wt)) return fail(ARD_EINVAL, "BWD_DATA needs dYin and Wt");
    if (a.mode == ARD_CONV_BWD_WEIGHT && (!dYin || !A)) return fail(ARD_EINVAL, "BWD_WEIGHT needs dYin and A");
    if (a.mode >= ARD_CONV_FWD && a.mode <= ARD_CONV_BWD_WEIGHT) return conv_run_planes(a, A, Wt, dYin, out, d_keep, w, stream);
  }

  if (a.mode == ARD_CONV_FWD) {
    if (!A || !Wt) return fail(ARD_EINVAL, "FWD needs A and Wt");
    if (Ck == 0) return fill_matrix(a.dtype, out, (long)a.N * a.Cout * a.Ho * a.Wo, 0.0f, stream);
    const long total = (long)a.Cout * taps * Ck;
    ARD_LAUNCH(pack_weights_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       (const T*)Wt, (const int*)d_keep, a.C, taps, a.Cout, Ck, 0, (T*)w.wp);
    ARD_LAUNCH_CHECK("pack_weights_kernel");
    ConvGemmParams P{};
    P.K = taps * Ck;
    P.Wp = Operand{w.wp, P.K, axis_identity(a.Cout), (P.K % ce) == 0};
    P.src = A;
    P.g = ConvGeom{a.N, a.C, a.H, a.W, a.Ho, a.Wo, a.kh, a.kw, a.stride, a.pad, a.pad, Ck, d_keep};
    if (a.blk) {
      P.g.blk = a.blk;
      P.g.bx = a.bx, P.g.by = a.by;
      P.g.RB = ceil_div(a.Ho * a.Wo, a.bx), P.g.CB = ceil_div(a.C * taps, a.by);
    }
    P.M = a.Cout;
    P.Ncols = (long)a.N * a.Ho * a.Wo;
    P.C.p = out;
    P.C.rm = axis_identity(a.Cout);
    P.C.cn = axis_identity((int)P.Ncols);
    P.C.plane = a.Ho * a.Wo;
    P.C.img_stride = (long)a.Cout * a.Ho * a.Wo;
    P.C.alpha = 1.0f;
    P.tiles_n = ceil_div((int)P.Ncols, 128);
    long blocks = (long)ceil_div(P.M, 128) * P.tiles_n;
    ARD_LAUNCH((conv_gemm_kernel<T, 128, 128, 2, 2>), dim3((unsigned)blocks), dim3(256), 0, stream, P);
    ARD_LAUNCH_CHECK("conv_gemm_kernel");
    return ARD_OK;
  }

  if (a.mode == ARD_CONV_BWD_DATA) {
    if (!dYin || !Wt) return fail(ARD_EINVAL, "BWD_DATA needs dYin and Wt");
    if (a.stride != 1) return fail(ARD_EUNSUPPORTED, "BWD_DATA is built for stride 1 only (got %d)", a.stride);
    if (a.kh - 1 - a.pad < 0 || a.kw - 1 - a.pad < 0) return fail(ARD_EUNSUPPORTED, "BWD_DATA needs pad <= k-1");
    if (Ck == 0) return fill_matrix(a.dtype, out, (long)a.N * a.C * a.H * a.W, 0.0f, stream);
    const long total = (long)Ck * taps * a.Cout;
    ARD_LAUNCH(pack_weights_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       (const T*)Wt, (const int*)d_keep, a.C, taps, Ck, a.Cout, 1, (T*)w.wp);
    ARD_LAUNCH_CHECK("pack_weights_kernel");
    ConvGemmParams P{};
    P.K = taps * a.Cout;
    P.Wp = Operand{w.wp, P.K, axis_identity(Ck), (P.K % ce) == 0};
    P.src = dYin;
    P.g = ConvGeom{a.N, a.Cout, a.Ho, a.Wo, a.H, a.W, a.kh, a.kw, 1, a.kh - 1 - a.pad, a.kw - 1 - a.pad, a.Cout, nullptr};
    if (a.blk) {
      P.Wp.vec = (a.Cout % ce) == 0;  // the contraction is walked tap by tap: every tap must start on a chunk
      P.g.blk = a.blk;
      P.g.bx = a.bx, P.g.by = a.by;
      P.g.RB = ceil_div(a.Ho * a.Wo, a.bx), P.g.CB = ceil_div(a.C * taps, a.by);
    }
    P.M = Ck;
    P.Ncols = (long)a.N * a.H * a.W;
    P.C.p = out;
    P.C.rm = axis_list(d_keep, Ck, a.C);
    P.C.cn = axis_identity((int)P.Ncols);
    P.C.plane = a.H * a.W;
    P.C.img_stride = (long)a.C * a.H * a.W;
    P.C.fill = a.kept_only ? 0 : 1;
    P.C.alpha = 1.0f;
    P.tiles_n = ceil_div((int)P.Ncols, 128);
    long blocks = (long)ceil_div(P.M, 128) * P.tiles_n;
    if (a.blk) {
      ARD_LAUNCH((conv_bwd_data_blocks_kernel<T, 128, 128, 2, 2>), dim3((unsigned)blocks), dim3(256), 0, stream, P);
      ARD_LAUNCH_CHECK("conv_bwd_data_blocks_kernel");
      return ARD_OK;
    }
    ARD_LAUNCH((conv_gemm_kernel<T, 128, 128, 2, 2>), dim3((unsigned)blocks), dim3(256), 0, stream, P);
    ARD_LAUNCH_CHECK("conv_gemm_kernel");
    return ARD_OK;
  }

  if (a.mode == ARD_CONV_BWD_WEIGHT) {
    if (!dYin || !A) return fail(ARD_EINVAL, "BWD_WEIGHT needs dYin and A");
    if (Ck == 0) return fill_matrix(a.dtype, out, (long)a.Cout * a.C * taps, 0.0f, stream);
    ARD_LAUNCH(rank_from_keep_kernel, dim3(1), dim3(1024), 0, stream, (const int*)d_keep, Ck, a.C, w.rank);
    ARD_LAUNCH_CHECK("rank_from_keep_kernel");
    ConvWgradParams P{};
    P.dY = dYin;
    P.A = A;
    P.g = ConvGeom{a.N, a.C, a.H, a.W, a.Ho, a.Wo, a.kh, a.kw, a.stride, a.pad, a.pad, Ck, d_keep};
    if (a.blk) {
      P.g.blk = a.blk;
      P.g.bx = a.bx, P.g.by = a.by;
      P.g.RB = ceil_div(a.Ho * a.Wo, a.bx), P.g.CB = ceil_div(a.C * taps, a.by);
    }
    P.part = w.part;
    P.Cout = a.Cout;
    P.Nn = Ck * taps;
    P.K = (long)a.N * a.Ho * a.Wo;
    const int hw = a.Ho * a.Wo;
    P.dy_vec = (hw % ce) == 0 && al16c(dYin);
    const int bk = 8 * ce;
    int splits = w.splits;
    long per = (P.K + splits - 1) / splits;
    per = (per + bk - 1) / bk * bk;
    splits = (int)((P.K + per - 1) / per);
    P.k_per_split = (int)per;
    P.tiles_n = ceil_div(P.Nn, 128);
    dim3 grid((unsigned)(ceil_div(P.Cout, 128) * P.tiles_n), (unsigned)splits);
    ARD_LAUNCH((conv_wgrad_kernel<T, 128, 128, 2, 2>), grid, dim3(256), 0, stream, P);
    ARD_LAUNCH_CHECK("conv_wgrad_kernel");
    const long total = (long)a.Cout * a.C * taps;
    ARD_LAUNCH(conv_wgrad_reduce_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       (const float*)w.part, (const int*)w.rank, splits, a.Cout, a.C, taps, P.Nn, a.kept_only, (T*)out);
    ARD_LAUNCH_CHECK("conv_wgrad_reduce_kernel");
    return ARD_OK;
  }
  return fail(ARD_EINVAL, "unknown conv mode %d", a.mode);
}

}  // namespace ard

using namespace ard;

extern "C" int32_t ard_conv_out_size(int32_t in, int32_t k, int32_t stride, int32_t pad) {
  if (in <= 0 || k <= 0 || stride <= 0 || pad < 0) return fail(ARD_ESHAPE, "non-positive convolution size");
  if (in + 2 * pad < k) return fail(ARD_ESHAPE, "kernel larger than the padded input");
  return (in + 2 * pad - k) / stride + 1;
}

extern "C" size_t ard_conv_workspace_bytes(int32_t dtype, int32_t N, int32_t C, int32_t H, int32_t Wd, int32_t Cout,
                                           int32_t kh, int32_t kw, int32_t stride, int32_t pad) {
  ConvArgs a{0, dtype, N, C, H, Wd, Cout, kh, kw, stride, pad, 0, 0, 0, 0, 0};
  if (conv_check(a)) return 0;
  return conv_ws_layout(nullptr, a).total;
}

extern "C" int32_t ard_conv_fwd_blocks(int32_t dtype, int32_t N, int32_t C, int32_t H, int32_t Wd, int32_t Cout, int32_t kh,
                                       int32_t kw, int32_t stride, int32_t pad, int32_t x, int32_t y, const void* A,
                                       const void* Wt, const uint8_t* d_block_keep, void* out, void* ws, size_t ws_bytes,
                                       void* stream) {
  BatchSuspend not_recorded;
  ConvArgs a{ARD_CONV_FWD, dtype, N, C, H, Wd, Cout, kh, kw, stride, pad, C, 0, 0, 0, 0, d_block_keep, x, y};
  int32_t st = conv_check(a);
  if (st) return st;
  if (x < 1 || y < 0) return fail(ARD_EINVAL, "block size must be positive (y = 0: the whole width)");
  if (y == 0) a.by = C * kh * kw;
  if (!A || !Wt || !d_block_keep || !out) return fail(ARD_EINVAL, "null pointer");
  ConvWs w = conv_ws_layout((char*)ws, a);
  if (!ws || ws_bytes < w.total) return fail(ARD_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", w.total, ws_bytes);
  if (dtype == ARD_BF16)
    return conv_run<uint16_t>(a, 0.0, A, Wt, nullptr, out, nullptr, nullptr, nullptr, nullptr, w, (hipStream_t)stream);
  // fp32 blocks of whole channels, as in the backward passes: per column block the fast pass over its channels alone, of
  // which the positions of kept bands are added.  The patch loaders of the general engine took 165 us and more for the
  // smallest layers; 24 drawn ones of 1 to 4 column blocks 1.6 to 13 times as fast (8 x 64 channels of 16 x 16 -> 16
  // 165 -> 12 us, 96 x 256 of 27 x 27 -> 32 1401 -> 273, 75 x 64 of 16 x 16 -> 330 232 -> 148).
  // Many blocks of few channels are the general engine's: a block is three launches, reads and writes the result once more and fills up
  // to 16 channels (36 x 16 of 19 x 19 -> 2, 1 x 1, a channel each: 17 against 182 us).  Times of both in us, fitted to 1500
  // layers of 1 to 16 blocks: within 0.3 % of the faster one in the mean over 400 others.
  const int taps = kh * kw, CB = ceil_div(C * taps, a.by), RB = ceil_div(a.Ho * a.Wo, x), cpb = a.by / taps;
  const double npix = (double)N * a.Ho * a.Wo, held = (double)CB * pad16(cpb), tiles = (double)ceil_div(Cout, 128) * ((npix + 127.0) / 128.0);
  const double passes_us = 1.7 + 10.0 * CB + 4.7e-6 * (CB - 0.25) * npix * Cout + 2.5e-6 * held * npix + 2.67e-8 * held * taps * npix * imax(Cout, 32) +
                           2.2e-3 * held * taps;
  const int steps = ceil_div(C * taps, 32);
  const double patches_us = 4.6 + (tiles > 256.0 ? tiles / 256.0 : 1.0) * (8.34 * steps + 8.25) + imin(Cout, 128) / 128.0 * (0.41 * steps + 20.0);
  if (w.plane_a && !dev_knobs().no_fast && a.by % taps == 0 && CB <= 16 && N <= 65535 && passes_us <= patches_us) {
    hipStream_t s = (hipStream_t)stream;
    ARD_LAUNCH(iota_kernel, dim3(ceil_div(C, 256)), dim3(256), 0, s, w.all_chan, C);
    ARD_LAUNCH_CHECK("iota_kernel");
    for (int cb = 0; cb < CB; ++cb) {
      ConvArgs g = a;
      g.blk = nullptr;
      g.n_keep = (cb + 1) * cpb <= C ? cpb : C - cb * cpb;
      st = conv_run<float>(g, 0.0, A, Wt, nullptr, w.dy_rows, nullptr, w.all_chan + cb * cpb, nullptr, nullptr, w, s);
      if (st) return st;
      ARD_LAUNCH(add_bands_kernel, dim3(Cout, N), dim3(256), 0, s, (const float*)w.dy_rows, d_block_keep, RB, CB, cb, x, fast_div((uint32_t)x), Cout,
                 a.Ho * a.Wo, (float*)out);
      ARD_LAUNCH_CHECK("add_bands_kernel");
    }
    return ARD_OK;
  }
  return conv_run<float>(a, 0.0, A, Wt, nullptr, out, nullptr, nullptr, nullptr, nullptr, w, (hipStream_t)stream);
}

extern "C" int32_t ard_conv_bwd_blocks(int32_t mode, int32_t dtype, int32_t N, int32_t C, int32_t H, int32_t Wd, int32_t Cout,
                                       int32_t kh, int32_t kw, int32_t stride, int32_t pad, int32_t x, int32_t y,
                                       const void* A, const void* Wt, const void* dYin, const uint8_t* d_block_keep, void* out,
                                       void* ws, size_t ws_bytes, void* stream) {
  BatchSuspend not_recorded;
  const int32_t reuse = mode & ARD_CONV_REUSE_DY;
  mode &= ~ARD_CONV_REUSE_DY;
  if ((mode != ARD_CONV_BWD_DATA && mode != ARD_CONV_BWD_WEIGHT) || (reuse && mode != ARD_CONV_BWD_WEIGHT))
    return fail(ARD_EINVAL, "mode must be ARD_CONV_BWD_DATA or ARD_CONV_BWD_WEIGHT (got %d)", mode);
  ConvArgs a{mode, dtype, N, C, H, Wd, Cout, kh, kw, stride, pad, C, 0, 0, 0, 0, d_block_keep, x, y};
  int32_t st = conv_check(a);
  if (st) return st;
  if (x < 1 || y < 0) return fail(ARD_EINVAL, "block size must be positive (y = 0: the whole width)");
  if (y == 0) a.by = C * kh * kw;
  if (!dYin || !d_block_keep || !out) return fail(ARD_EINVAL, "null pointer");
  if (mode == ARD_CONV_BWD_WEIGHT && !A) return fail(ARD_EINVAL, "BWD_WEIGHT needs A");
  if (mode == ARD_CONV_BWD_DATA) {
    if (!Wt) return fail(ARD_EINVAL, "BWD_DATA needs Wt");
    if (stride != 1) return fail(ARD_EUNSUPPORTED, "BWD_DATA is built for stride 1 only (got %d)", stride);
    if (kh - 1 - pad < 0 || kw - 1 - pad < 0) return fail(ARD_EUNSUPPORTED, "BWD_DATA needs pad <= k-1");
  }
  ConvWs w = conv_ws_layout((char*)ws, a);
  if (!ws || ws_bytes < w.total) return fail(ARD_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", w.total, ws_bytes);
  hipStream_t s = (hipStream_t)stream;
  const int taps = kh * kw;
  const int CB = ceil_div(C * taps, a.by), RB = ceil_div(a.Ho * a.Wo, a.bx);
  // Groups of whole channels on the channels-last grids: the weight gradient contracts over the kept positions of each, all of
  // them in one launch; the data gradient is one launch over tiles of positions, or over the kept positions alone, whichever
  // is expected to be faster (22 images of 64 channels of 56 x 56 -> 24, 5 x 5, 30 % kept: 33 against 74 us; 56 of 64 of 56 x 56 -> 48,
  // 3 x 3: 39 and 50; 64 of 512 of 14 x 14 -> 512: 120 and 59).
  const bool by_groups = w.grid_a && !dev_knobs().no_fast && a.by % (8 * taps) == 0 && CB * (a.by / taps) <= pad64(C) && CB <= w.pos_blocks;
  ScatterDataParams sd;
  BlockDataParams bd{};
  int ks;
  const BandMask bands{d_block_keep, RB, CB, 0, a.bx};
  const bool tiles = by_groups && block_data_tiles(a, w, bd);
  const bool over_kept = a.by % (16 * taps) == 0 && scatter_plan(a, w, bands, a.by / taps, sd, ks) &&
                         (tiles ? scatter_us(sd, ks, kKeptGuess, a.bx) <= block_tiles_us(a, bd)
                                : CB > 1 || scatter_us(sd, ks, kKeptGuess, a.bx) <= masked_us(a) + 6.0);  // (masked passes: a launch more)
  const bool one_launch = over_kept || tiles;
  const bool listed = by_groups && pos_lists_fit(a);
  if (listed) a.lists = pos_list_job(a, d_block_keep, a.bx, CB, w);
  if (one_launch && mode == ARD_CONV_BWD_DATA) {
    if (!over_kept) return conv_block_data(a, bd, Wt, dYin, out, w, s);
    ConvArgs g = a;
    g.blk = nullptr;
    g.scatter = bands, g.scatter_cpb = a.by / taps;
    return conv_run<uint16_t>(g, 0.0, A, Wt, dYin, out, nullptr, nullptr, nullptr, nullptr, w, s);
  }
  if (listed && mode == ARD_CONV_BWD_WEIGHT) {
    ConvArgs g = a;
    g.blk = nullptr;
    g.cpb = a.by / taps;
    // (else the data gradient left dY masked for its last column block, or on a grid of another shape)
    g.reuse = one_launch || (CB == 1 && kh - 1 == 2 * pad && kw - 1 == 2 * pad) ? reuse : 0;
    return conv_run<uint16_t>(g, 0.0, A, Wt, dYin, out, nullptr, nullptr, nullptr, nullptr, w, s);
  }
  const PosListJob lists = a.lists;
  a.lists = PosListJob{};
  // every channel is kept: the passes take the identity list
  ARD_LAUNCH(iota_kernel, dim3(ceil_div(C, 256)), dim3(256), 0, s, w.all_chan, C);
  ARD_LAUNCH_CHECK("iota_kernel");
  // Blocks of whole channels (y a multiple of kh*kw), not too many of them: column block cb is the channel
  // range [cb*cpb, (cb+1)*cpb) over all taps, and whether a term of those channels counts depends on the band
  // of the output position alone.  Per column block: dY copied with the positions of its dropped bands zeroed,
  // then the ordinary gradient pass (whichever engine takes the shape) with that channel range as the kept
  // list, writing its channels' part of the output only.  Work is not skipped, but the passes are the fast ones.
  if (a.by % taps == 0 && CB <= 16 && !(mode == ARD_CONV_BWD_DATA && stride != 1)) {
    const int cpb = a.by / taps;
    for (int cb = 0; cb < CB; ++cb) {
      ConvArgs g = a;
      g.blk = nullptr;
      g.kept_only = 1;
      g.n_keep = (cb + 1) * cpb <= C ? cpb : C - cb * cpb;
      const void* dy_use = w.dy_rows;
      if ((w.grid_a || w.plane_a) && !dev_knobs().no_fast) {
        // the pass copies dY into its grid anyway: that copy applies the mask
        g.dy_mask = BandMask{d_block_keep, RB, CB, cb, a.bx};
        dy_use = dYin;
        if (CB == 1) g.lists = lists;  // (for the weight gradient of the same workspace)
      } else {
        if (dtype == ARD_BF16)
          ARD_LAUNCH(mask_bands_kernel<uint16_t>, dim3(Cout, N), dim3(256), 0, s, (const uint16_t*)dYin, d_block_keep, RB, CB, cb,
                     a.bx, Cout, a.Ho * a.Wo, (uint16_t*)w.dy_rows);
        else
          ARD_LAUNCH(mask_bands_kernel<float>, dim3(Cout, N), dim3(256), 0, s, (const float*)dYin, d_block_keep, RB, CB, cb, a.bx,
                     Cout, a.Ho * a.Wo, (float*)w.dy_rows);
        ARD_LAUNCH_CHECK("mask_bands_kernel");
      }
      st = dtype == ARD_BF16 ? conv_run<uint16_t>(g, 0.0, A, Wt, dy_use, out, nullptr, w.all_chan + cb * cpb, nullptr, nullptr, w, s)
                             : conv_run<float>(g, 0.0, A, Wt, dy_use, out, nullptr, w.all_chan + cb * cpb, nullptr, nullptr, w, s);
      if (st) return st;
    }
    return ARD_OK;
  }
  if (dtype == ARD_BF16)
    return conv_run<uint16_t>(a, 0.0, A, Wt, dYin, out, nullptr, w.all_chan, nullptr, nullptr, w, s);
  return conv_run<float>(a, 0.0, A, Wt, dYin, out, nullptr, w.all_chan, nullptr, nullptr, w, s);
}

extern "C" int32_t ard_fmap_drop_conv(int32_t mode, int32_t dtype, int32_t N, int32_t C, int32_t H, int32_t Wd,
                                      int32_t Cout, int32_t kh, int32_t kw, int32_t stride, int32_t pad, double rate,
                                      int32_t n_keep, const void* A, const void* Wt, const void* dYin, void* out,
                                      uint8_t* d_mask, int32_t* d_keep, int32_t* d_count, int64_t* d_score, void* ws,
                                      size_t ws_bytes, void* stream) {
  BatchSuspend not_recorded;  // this entry point's kernels depend on each other: never part of a grouped launch
  const int32_t pad_keep = (mode & 0xff) == ARD_CONV_SELECT && (mode & ARD_CONV_PAD_KEEP) ? 1 : 0;
  if (pad_keep) mode &= ~ARD_CONV_PAD_KEEP;
  if (mode < 0 || (mode & ~(0xff | ARD_CONV_REUSE_A | ARD_CONV_REUSE_DY))) return fail(ARD_EINVAL, "unknown conv mode bits 0x%x", mode);
  ConvArgs a{mode & 0xff, dtype, N, C, H, Wd, Cout, kh, kw, stride, pad, n_keep, 0, 0, 0, mode & (ARD_CONV_REUSE_A | ARD_CONV_REUSE_DY)};
  a.pad_keep = pad_keep;
  if (a.reuse && a.mode == ARD_CONV_SELECT) return fail(ARD_EINVAL, "SELECT builds no grid");
  int32_t st = conv_check(a);
  if (st) return st;
  ConvWs w = conv_ws_layout((char*)ws, a);
  if (!ws || ws_bytes < w.total)
    return fail(ARD_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", w.total, ws_bytes);
  if (dtype == ARD_BF16)
    return conv_run<uint16_t>(a, rate, A, Wt, dYin, out, d_mask, d_keep, d_count, d_score, w, (hipStream_t)stream);
  return conv_run<float>(a, rate, A, Wt, dYin, out, d_mask, d_keep, d_count, d_score, w, (hipStream_t)stream);
}
