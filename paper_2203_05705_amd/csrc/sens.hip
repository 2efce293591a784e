// Region-level sensitivity prediction and the sensitivity-aware dropout patterns of the CNN variant
// (Sections 5.1, 5.2.1, 5.2.2): which rows (output positions) or blocks of a layer's input matrix are
// dropped in this iteration.
//
// The input matrix of an image has one row per output position p = oh * Wo + ow and one column per
// (c, kh, kw), q = (c * KH + kh) * KW + kw, entry = zero-padded A[c, oh*s + kh - pad, ow*s + kw - pad];
// it is never built: the kernels address the activations directly.  It is cut into x-by-y regions
// (row band rb = p / x, column block cb = q / y, edge regions clipped).
//
// Every random draw is a 32-bit word of the SplitMix64 finaliser chained over
// (seed, iteration, stream, index) -- stateless and integer only, so the masks are reproducible bit for
// bit on any number of devices (the host folds the first three links, the kernels add the index).
#include <math.h>

#include <type_traits>

#include "common.hpp"

namespace ard {

static __host__ __device__ inline uint64_t sens_mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}
constexpr uint64_t kSensGolden = 0x9E3779B97F4A7C15ULL;
enum { SENS_STREAM_SAMPLE = 0x5E01, SENS_STREAM_ROWS = 0x5E02, SENS_STREAM_BLOCKS = 0x5E03 };

static uint64_t sens_prefix(uint64_t seed, uint64_t iter, uint32_t stream) {
  uint64_t h = sens_mix64(seed + kSensGolden);
  h = sens_mix64((h ^ iter) + kSensGolden);
  return sens_mix64((h ^ (uint64_t)stream) + kSensGolden);
}
static __device__ __forceinline__ uint32_t sens_draw(uint64_t prefix, uint64_t index) {
  return (uint32_t)(sens_mix64((prefix ^ index) + kSensGolden) >> 32);
}
static uint64_t sens_threshold(double p) {
  double q = floor(p * 4294967296.0);
  if (q < 0) q = 0;
  if (q > 4294967296.0) q = 4294967296.0;
  return (uint64_t)q;
}

struct SensGeom {
  int N, C, H, W, KH, KW, stride, pad, Ho, Wo;
  int rows, cols;  // of the input matrix of one image
  int x, y, RB, CB;
};

// One workgroup per (image, region): s = max(1, k * size / 1000) draws with replacement, count of the
// drawn entries above the threshold (Section 5.1, steps 2 and 3).
template <typename T>
__global__ __launch_bounds__(256) void sens_predict_kernel(const T* A, SensGeom g, int k_permille, int t_permille, float thr,
                                                           uint64_t prefix, int* count, int* samples, uint8_t* sens) {
  __shared__ int wave_cnt[4];
  const int region = blockIdx.x;  // (image * RB + rb) * CB + cb
  const int cb = region % g.CB, rb = (region / g.CB) % g.RB, n = region / (g.CB * g.RB);
  const int r0 = rb * g.x, q0 = cb * g.y;
  const int h = min(g.x, g.rows - r0), w = min(g.y, g.cols - q0);
  const int size = h * w;
  int s = (int)(((long)k_permille * size) / 1000);
  if (s < 1) s = 1;
  const T* img = A + (long)n * g.C * g.H * g.W;
  const int taps = g.KH * g.KW;
  int c = 0;
  for (int j = threadIdx.x; j < s; j += 256) {
    const uint32_t u = sens_draw(prefix, (uint64_t)region * 65536u + (uint64_t)j);
    const int e = (int)(((uint64_t)u * (uint64_t)size) >> 32);
    const int p = r0 + e / w, q = q0 + e % w;
    const int oh = p / g.Wo, ow = p - oh * g.Wo;
    const int ch = q / taps, tap = q - ch * taps;
    const int kh = tap / g.KW, kw = tap - kh * g.KW;
    const int ih = oh * g.stride + kh - g.pad, iw = ow * g.stride + kw - g.pad;
    float v = 0.0f;  // the zero border of the input matrix
    if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W) v = ElemTraits<T>::to_f32(img[((long)ch * g.H + ih) * g.W + iw]);
    c += v > thr ? 1 : 0;
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  if ((threadIdx.x & 63) == 0) wave_cnt[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int tot = wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
    count[region] = tot;
    samples[region] = s;
    sens[region] = (1000L * tot >= (long)t_permille * s) ? 1 : 0;
  }
}

// The same prediction with the region's geometry tabulated in LDS once per workgroup: per column of the
// region its channel's offset in the image and its tap (kh, kw), per row of the band its top-left input
// position.  A draw is then the mixer, one division by the region's width, two LDS reads and the gather.
// Same draws, same elements, same counts as sens_predict_kernel (bit for bit); used when the table fits
// (region width <= kSensLutCols, channel offsets below 2^24, taps below 16).
constexpr int kSensLutCols = 8192, kSensLutRows = 1024;
template <typename T>
__global__ __launch_bounds__(256) void sens_predict_lut_kernel(const T* A, SensGeom g, int k_permille, int t_permille, float thr,
                                                               uint64_t prefix, FastDiv div_w, int* count, int* samples,
                                                               uint8_t* sens) {
  extern __shared__ int sens_lut[];  // [w] columns, then [h] rows
  __shared__ int wave_cnt[4];
  const int region = blockIdx.x;  // (image * RB + rb) * CB + cb
  const int cb = region % g.CB, rb = (region / g.CB) % g.RB, n = region / (g.CB * g.RB);
  const int r0 = rb * g.x, q0 = cb * g.y;
  const int h = min(g.x, g.rows - r0), w = min(g.y, g.cols - q0);
  const int size = h * w;
  int s = (int)(((long)k_permille * size) / 1000);
  if (s < 1) s = 1;
  const int taps = g.KH * g.KW;
  int* col_lut = sens_lut;
  int* row_lut = sens_lut + w;
  for (int i = threadIdx.x; i < w; i += 256) {
    const int q = q0 + i;
    const int ch = q / taps, tap = q - ch * taps;
    const int kh = tap / g.KW, kw = tap - kh * g.KW;
    col_lut[i] = (ch * g.H * g.W) | (kh << 24) | (kw << 28);
  }
  for (int i = threadIdx.x; i < h; i += 256) {
    const int p = r0 + i;
    const int oh = p / g.Wo, ow = p - oh * g.Wo;
    // input position of tap (0, 0), biased by the padding so that both halves are non-negative
    row_lut[i] = (oh * g.stride) | ((ow * g.stride) << 16);
  }
  __syncthreads();
  const T* img = A + (long)n * g.C * g.H * g.W;
  int c = 0;
  for (int j = threadIdx.x; j < s; j += 256) {
    const uint32_t u = sens_draw(prefix, (uint64_t)region * 65536u + (uint64_t)j);
    const uint32_t e = (uint32_t)(((uint64_t)u * (uint64_t)size) >> 32);
    const uint32_t r = fdiv(e, div_w), q = e - r * (uint32_t)w;
    const int ci = col_lut[q], ri = row_lut[r];
    const int ih = (ri & 0xffff) + ((ci >> 24) & 15) - g.pad, iw = (ri >> 16) + ((ci >> 28) & 15) - g.pad;
    float v = 0.0f;  // the zero border of the input matrix
    if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W) v = ElemTraits<T>::to_f32(img[(ci & 0xffffff) + ih * g.W + iw]);
    c += v > thr ? 1 : 0;
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  if ((threadIdx.x & 63) == 0) wave_cnt[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int tot = wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
    count[region] = tot;
    samples[region] = s;
    sens[region] = (1000L * tot >= (long)t_permille * s) ? 1 : 0;
  }
}

// The prediction once more, with the footprint of the workgroup's regions in the activations brought into LDS
// first: the draws of a region fall on a few input rows of its channels (a band of 8 positions of a 28 x 28 layer of 256
// channels: 4 rows x 28 x 256 for 5529 draws), and a gather from memory costs a whole cache-line transaction per
// draw.  Same draws, same elements, same counts.
//
// What a draw needs of an element is one bit (above the threshold or not).  The bits of a row of W + 2 pad, with the
// zero border of the input matrix around them, are whole words, so that a draw's bit number is a sum of one table entry
// for its row and one for its column, nothing is tested, and a thread makes a word of a row out of at most five loads
// and stores it once.  (Where rows shared words, 16-byte pieces were cut at the row ends and added with atomics: with the
// copies of 14 workgroups per image, of four rows for two, 46 of the pass's 97 us.)
//
// Then the pass is bound by the vector instructions of a draw (leaving out its LDS reads changes nothing; a multiplication
// costs 2.0 ns of a SIMD, as any instruction of eight bytes does, one of four bytes 1.2), and saves what it can of them:
//  * the bits of (prefix ^ index) + golden above the lowest 16 take two values over a region (j < 65536; the sum
//    carries or it does not).  Thread t of four wavefronts takes the draws whose index is t ^ (low byte of prefix) in its
//    lowest byte, i.e. t + golden is what this byte becomes before its carry, and the next byte i is the same for all
//    threads: the mixer's first product is a number of the thread's (one of two) plus one that depends on i, which a
//    wavefront tabulates in its lanes and reads back as a scalar.  Only the last 21 threads' bytes carry into i's: their
//    wavefront makes both tables.
//  * only the upper half of the second product is needed;
//  * u * h = (row, f) and f * w = (column, .) give row and column of the drawn element without dividing.
// N=128, 256 channels, 28x28, 3x3, 30 % sampled (69 M draws): bands of 8 positions 99 -> 88 us with the activations in the
// Infinity Cache and 98 -> 92 from memory, 112 x 576 regions 83 -> 78 and 84 -> 84 (all workgroups copy first, and then all
// draw); over 60 layers (8 - 128 images, 16 - 512 channels, 7 x 7 - 56 x 56, both types) 1.17x in the geometric mean.
// Workgroups of 8 and 4 wavefronts: 92 and 93, 85 and 86 us; twice and four times as many: 93 and 97, 87 and 91 from memory.
struct SensStage {
  int nrow, words;        // staged rows of a channel (border included), words of a row
  FastDiv div_taps, div_kw, div_wo, div_words, div_items;  // ... words of a row, of a channel
  int G, RBG;             // consecutive row bands (of one image and column block) per workgroup; groups per image
};
constexpr int kSensWaves = 16;
struct SensBand {  // what the draws of a band share, made once by a thread of its own
  uint64_t K[2];
  uint32_t m[2], p16;
  int s, h, hits, pad[2];
};
static_assert(sizeof(SensBand) == 48, "whole 16-byte pieces");
// element > threshold shifted into b from below
__device__ __forceinline__ void sens_push(uint32_t& b, float v, float thr) {
  asm("v_cmp_gt_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(b) : "v"(v), "v"(thr) : "vcc");
}
typedef uint32_t sens_u32x4 __attribute__((ext_vector_type(4), aligned(4)));
// bits of the `n` <= 32 elements from A[first] on, lowest first (whatever lies above them is to be masked off); `end`: elements
// of the tensor
__device__ __forceinline__ uint32_t sens_word(const uint16_t* A, long first, int n, int most, long end, float thr) {
  const long d0 = first >> 1;
  const int odd = (int)(first & 1), quads = (most + 8) >> 3;  // (uniform: for the longest word, first element odd)
  uint32_t b = 0;
  if (d0 + 4 * quads <= end >> 1) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(A) + d0;
    sens_u32x4 v[5];
#pragma unroll
    for (int q = 0; q < 5; ++q)
      if (q < quads) v[q] = *reinterpret_cast<const sens_u32x4*>(src + 4 * q);
#pragma unroll
    for (int q = 4; q >= 0; --q) {
      if (q >= quads) continue;
#pragma unroll
      for (int e = 3; e >= 0; --e) {
        sens_push(b, __uint_as_float(v[q][e] & 0xffff0000u), thr);
        const uint32_t above = b;
        sens_push(b, __uint_as_float(v[q][e] << 16), thr);
        if (q == 0 && e == 0 && odd) b = above;
      }
    }
  } else {
    for (int e = n - 1; e >= 0; --e) sens_push(b, bf16_bits_to_f32(A[first + e]), thr);
  }
  return b;
}
__device__ __forceinline__ uint32_t sens_word(const float* A, long first, int n, int most, long end, float thr) {
  uint32_t b = 0;
  if (first + ((most + 15) & ~15) <= end) {
#pragma unroll 1
    for (int o = (most - 1) & ~15; o >= 0; o -= 16) {  // (sixteen registers at a time)
      sens_u32x4 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const sens_u32x4*>(A + first + o + 4 * q);
#pragma unroll
      for (int q = 3; q >= 0; --q)
#pragma unroll
        for (int e = 3; e >= 0; --e) sens_push(b, __uint_as_float(v[q][e]), thr);
    }
  } else {
    for (int e = n - 1; e >= 0; --e) sens_push(b, A[first + e], thr);
  }
  return b;
}
template <typename T>
__global__ __launch_bounds__(64 * kSensWaves, 8) void sens_predict_staged_kernel(const T* A, SensGeom g, SensStage sg, int k_permille,
                                                                                 int t_permille, float thr, uint64_t prefix,
                                                                                 int* count, int* samples, uint8_t* sens) {
  extern __shared__ uint4 sens_stage_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NT = 64 * kSensWaves;
  // workgroup = (image, group of G row bands, column block)
  const int cb = blockIdx.x % g.CB, rbg = (blockIdx.x / g.CB) % sg.RBG, n = blockIdx.x / (g.CB * sg.RBG);
  const int rb_first = rbg * sg.G, nb = min(sg.G, g.RB - rb_first);
  if (nb <= 0) return;
  const int r0 = rb_first * g.x, q0 = cb * g.y;
  const int h = min(nb * g.x, g.rows - r0), w = min(g.y, g.cols - q0);  // rows of the group, columns of the block
  const int taps = g.KH * g.KW, pitch = sg.words * 32, ch_bits = sg.nrow * pitch;
  // footprint: channels [ch_lo, ch_hi], sg.nrow input rows from `top` on (border included)
  const int ch_lo = q0 / taps, ch_hi = (q0 + w - 1) / taps;
  const int oh_lo = r0 / g.Wo, top = oh_lo * g.stride - g.pad;
  const int nch = ch_hi - ch_lo + 1, items = nch * sg.nrow * sg.words;
  uint32_t* bits = reinterpret_cast<uint32_t*>(sens_stage_lds + 3 * sg.G);
  int* col_lut = reinterpret_cast<int*>(bits + items);
  int* row_lut = col_lut + w;
  SensBand* bands = reinterpret_cast<SensBand*>(sens_stage_lds);  // (first: aligned)
  const int border_above = 0.0f > thr ? 1 : 0;  // the zero border: bits are kept relative to it
  const long img = (long)n * g.C * g.H * g.W, end = (long)g.N * g.C * g.H * g.W;
  for (int i = tid; i < items; i += NT) {
    const int c = (int)fdiv((uint32_t)i, sg.div_items), rw = i - c * sg.nrow * sg.words;
    const int r = (int)fdiv((uint32_t)rw, sg.div_words), x0 = (rw - r * sg.words) * 32 - g.pad, ih = top + r;
    const int lo = max(x0, 0), len = min(x0 + 32, g.W) - lo;
    uint32_t b = 0;
    if (ih >= 0 && ih < g.H && len > 0) {
      b = sens_word(A, img + ((long)(ch_lo + c) * g.H + ih) * g.W + lo, len, min(g.W, 32), end, thr);
      if (border_above) b = ~b;
      b = (len < 32 ? b & ((1u << len) - 1u) : b) << (lo - x0);
    }
    bits[i] = b;
  }
  for (int i = tid; i < w; i += NT) {
    const int q = q0 + i;
    const int ch = (int)fdiv((uint32_t)q, sg.div_taps), tap = q - ch * taps;
    const int kh = (int)fdiv((uint32_t)tap, sg.div_kw), kw = tap - kh * g.KW;
    col_lut[i] = (ch - ch_lo) * ch_bits + kh * pitch + kw;
  }
  for (int i = tid; i < h; i += NT) {
    const int p = r0 + i;
    const int oh = (int)fdiv((uint32_t)p, sg.div_wo), ow = p - oh * g.Wo;
    row_lut[i] = (oh - oh_lo) * g.stride * pitch + ow * g.stride;
  }
  constexpr uint32_t C1L = 0x1CE4E5B9u, C1H = 0xBF58476Du, C2L = 0x133111EBu, C2H = 0x94D049BBu;
  constexpr uint64_t C1 = ((uint64_t)C1H << 32) | C1L;
  constexpr uint32_t g16 = (uint32_t)(kSensGolden & 0xffffu);
  for (int i = NT - 1 - tid; i < nb; i += NT) {
    SensBand v{};
    v.h = min(g.x, h - i * g.x);
    v.s = max(1, (int)(((long)k_permille * v.h * w) / 1000));
    // z = (prefix ^ index) + golden, index = region * 65536 + j: its bits from 16 up, without and with the carry
    const uint64_t P = prefix ^ ((uint64_t)(((n * g.RB) + rb_first + i) * g.CB + cb) << 16);
    for (int cy = 0; cy < 2; ++cy) {
      const uint64_t H = ((P >> 16) + (kSensGolden >> 16) + cy) & 0xffffffffffffULL;
      v.m[cy] = (uint32_t)(H >> 14) & 0xffffu;  // what z >> 30 puts on the lowest 16 bits
      v.K[cy] = ((H ^ (H >> 30)) << 16) * C1;
    }
    v.p16 = (uint32_t)P & 0xffffu;
    bands[i] = v;
  }
  __syncthreads();
  // A wavefront takes a quarter of the low bytes of one band at a time; of the bands beyond the last full round of the
  // workgroup it takes shares of the i, so that all wavefronts end together (rows of 8 positions: 7 rounds -> 6 and a part).
  constexpr int PER = kSensWaves / 4;  // bands of a round
  const int full = nb - nb % PER, jobs = (full + (nb - full) * PER) * 4;
  for (int job = wave; job < jobs; job += kSensWaves) {
    const int b4 = job >> 2, quarter = job & 3, part_of = b4 < full ? 1 : PER;
    const int band = b4 < full ? b4 : full + (b4 - full) / PER, chunk = b4 < full ? 0 : (b4 - full) % PER;
    const int* rows = row_lut + band * g.x;  // rows of this band within the group
    const SensBand& B = bands[band];
    const int s = __builtin_amdgcn_readfirstlane(B.s), hb = __builtin_amdgcn_readfirstlane(B.h), ni = (s + 255) >> 8;
    const int share = part_of == 1 ? ni : (ni + PER - 1) / PER, i_lo = chunk * share, i_hi = min(ni, i_lo + share);
    const uint64_t K0 = B.K[0], K1 = B.K[1];
    const uint32_t m0 = B.m[0], m1 = B.m[1], p16 = B.p16;
    const uint32_t t = (uint32_t)(quarter * 64 + lane), alo = t + (g16 & 255u), j_lo = t ^ (p16 & 255u);
    const bool c0 = alo > 255u;
    const uint64_t mine0 = (uint64_t)((alo ^ m0) & 255u) * C1, mine1 = (uint64_t)((alo ^ m1) & 255u) * C1;
    uint32_t c = 0;
    // the part of i = i0 + lane; bit l of cy: do the 16 bits of i0 + l carry?
    auto part = [&](int i, uint32_t carry, uint64_t& cy) {
      const uint32_t ahi = ((p16 >> 8) ^ (uint32_t)i) + (g16 >> 8) + carry;
      const bool over = ahi > 255u;
      cy = __ballot(over);
      return (over ? K1 : K0) + (((uint64_t)((ahi ^ ((over ? m1 : m0) >> 8)) & 255u) * C1) << 8);
    };
    auto lane64 = [](uint64_t v, int k) {
      return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), k) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)v, k);
    };
    auto place = [&](uint64_t y) {  // bit number of the draw whose first product is y
      uint32_t ylo = (uint32_t)y, yhi = (uint32_t)(y >> 32);
      ylo ^= (yhi << 5) | (ylo >> 27);
      yhi ^= yhi >> 27;
      uint32_t u = __umulhi(ylo, C2L) + ylo * C2H + yhi * C2L;
      u ^= u >> 31;
      const uint64_t uh = (uint64_t)u * (uint32_t)hb;
      return (uint32_t)rows[(uint32_t)(uh >> 32)] + (uint32_t)col_lut[__umulhi((uint32_t)uh, (uint32_t)w)];
    };
    auto share_of = [&](auto carries) {
      for (int i0 = i_lo; i0 < i_hi; i0 += 64) {
        const int e = min(64, i_hi - i0), whole = i0 + e > s >> 8 ? e - 1 : e;  // (the last i of a band may be a partial one)
        uint64_t cy0, cy1 = 0, S1 = 0;
        const uint64_t S0 = part(i0 + lane, 0, cy0);
        if constexpr (decltype(carries)::value) S1 = part(i0 + lane, 1, cy1);
        const uint64_t low_carries = __ballot(c0);
        auto at = [&](int k) {
          uint64_t S = lane64(S0, k), over;  // (which lanes' 16 bits carry: all alike but for low_carries)
          asm("s_bitcmp1_b64 %1, %2\n\ts_cselect_b64 %0, -1, 0" : "=s"(over) : "s"(cy0), "s"(k) : "scc");
          if constexpr (decltype(carries)::value) {
            uint64_t over1;
            asm("s_bitcmp1_b64 %1, %2\n\ts_cselect_b64 %0, -1, 0" : "=s"(over1) : "s"(cy1), "s"(k) : "scc");
            S = c0 ? lane64(S1, k) : S;
            over = (over & ~low_carries) | (over1 & low_carries);
          }
          uint32_t lo, hi;
          asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(lo) : "v"((uint32_t)mine0), "v"((uint32_t)mine1), "s"(over));
          asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(hi) : "v"((uint32_t)(mine0 >> 32)), "v"((uint32_t)(mine1 >> 32)), "s"(over));
          return place(S + (((uint64_t)hi << 32) | lo));
        };
        int k = 0;
        for (; k + 4 <= whole; k += 4) {  // (four draws in flight: their table and LDS reads overlap)
          uint32_t bit[4], word[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) bit[q] = at(k + q);
#pragma unroll
          for (int q = 0; q < 4; ++q) word[q] = bits[bit[q] >> 5];
#pragma unroll
          for (int q = 0; q < 4; ++q) c += __builtin_amdgcn_ubfe(word[q], bit[q], 1);
        }
        for (; k < e; ++k)
          if (k < whole || (int)j_lo < (s & 255)) {
            const uint32_t bit = at(k);
            c += __builtin_amdgcn_ubfe(bits[bit >> 5], bit, 1);
          }
      }
    };
    if (quarter < 3) share_of(std::integral_constant<bool, false>{});
    else share_of(std::integral_constant<bool, true>{});
    // sum over the wavefront, to its last lane
#define ARD_SENS_DPP(ctrl, rows) c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, ctrl, rows, 0xf, false)
    ARD_SENS_DPP(0x111, 0xf);  // 1, 2, 4, 8 lanes within a row of 16
    ARD_SENS_DPP(0x112, 0xf);
    ARD_SENS_DPP(0x114, 0xf);
    ARD_SENS_DPP(0x118, 0xf);
    ARD_SENS_DPP(0x142, 0xa);  // the rows before
    ARD_SENS_DPP(0x143, 0xc);
#undef ARD_SENS_DPP
    if (lane == 63) atomicAdd(&bands[band].hits, (int)c);
  }
  __syncthreads();
  for (int i = tid; i < nb; i += NT) {
    const int s = bands[i].s, tot = border_above ? s - bands[i].hits : bands[i].hits;
    const int region = ((n * g.RB) + rb_first + i) * g.CB + cb;
    count[region] = tot;
    samples[region] = s;
    sens[region] = (1000L * tot >= (long)t_permille * s) ? 1 : 0;
  }
}

// Row-based pattern (Section 5.2.1): global row g = image * rows + p is dropped iff its draw is below the
// possibility of its band (m if sensitive, n otherwise); mask (1 = kept) and ascending kept list by
// ballot + mbcnt compaction.  A workgroup takes `chunk` consecutive rows.  Where its part of the kept list
// starts is the number of kept rows before its chunk.  No scratch memory and no hand-over between
// workgroups: with a mask, a first launch (phase 0) writes it and the second (phase 1) counts its ones
// before the chunk with 16-byte loads; without one (phase 2, a single launch) the workgroup recounts the
// rows before its chunk -- a draw is a pure function of the row.
__global__ __launch_bounds__(1024) void sens_row_pattern_kernel(const uint8_t* sens, int n_rows_total, int rows, int x, int RB,
                                                               int CB, uint64_t tm, uint64_t tn, uint64_t prefix, int chunk,
                                                               int phase, uint8_t* mask, int* keep, int* count) {
  __shared__ int wave_tot[16];
  __shared__ int running_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int start = blockIdx.x * chunk, end = min(n_rows_total, start + chunk);
  auto row_kept = [&](int gr) {
    const int n = gr / rows, p = gr - n * rows;
    const bool sv = sens[((long)n * RB + p / x) * CB] != 0;  // (regions span the width: CB = 1)
    return !((uint64_t)sens_draw(prefix, (uint64_t)gr) < (sv ? tm : tn));
  };
  if (phase == 0) {
    for (int gr = start + tid; gr < end; gr += 1024) mask[gr] = row_kept(gr) ? 1 : 0;
    return;
  }
  int before = 0;
  if (phase == 1) {
    // ones of mask[0, start): start is a multiple of 1024, the mask 16-byte aligned (host checks)
    const uint4* m16 = reinterpret_cast<const uint4*>(mask);
    for (int i = tid; i < start / 16; i += 1024) {
      const uint4 v = m16[i];
      before += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
  } else {
    for (int gr = tid; gr < start; gr += 1024) before += row_kept(gr) ? 1 : 0;
  }
  for (int off = 32; off > 0; off >>= 1) before += __shfl_down(before, off, 64);
  if (lane == 0) wave_tot[wave] = before;
  __syncthreads();
  if (tid == 0) {
    int t = 0;
    for (int w = 0; w < 16; ++w) t += wave_tot[w];
    running_s = t;
  }
  __syncthreads();
  for (int base = start; base < end; base += 1024) {
    const int gr = base + tid;
    bool kept = false;
    if (gr < end) kept = phase == 1 ? mask[gr] != 0 : row_kept(gr);
    const unsigned long long bal = __ballot(kept);
    const int r = __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0));
    if (lane == 0) wave_tot[wave] = __popcll(bal);
    __syncthreads();
    int before_me = running_s, total = 0;
    for (int w = 0; w < 16; ++w) {
      const int t = wave_tot[w];
      if (w < wave) before_me += t;
      total += t;
    }
    if (kept && keep) keep[before_me + r] = gr;
    __syncthreads();
    if (tid == 0) running_s += total;
    __syncthreads();
  }
  if (tid == 0 && count && end == n_rows_total) *count = running_s;
}

// Block-based pattern (Section 5.2.2): one workgroup per (image, row band).  Balancing: S = mean number
// of sensitive blocks per band of this image, rounded half up; the S blocks of the band with the
// largest share count / samples (compared exactly by cross-multiplication, ties to the lower block)
// are the sensitive ones.  Then every block is dropped iff its draw is below m (sensitive) or n.
__global__ __launch_bounds__(256) void sens_block_pattern_kernel(const int* count, const int* samples, const uint8_t* sens,
                                                                 int RB, int CB, int balance, uint64_t tm, uint64_t tn,
                                                                 uint64_t prefix, uint8_t* sens_out, uint8_t* block_keep) {
  __shared__ int wave_sum[4];
  __shared__ int S_s;
  const int band = blockIdx.x;  // image * RB + rb
  const int n = band / RB;
  int tot = 0;
  for (int i = threadIdx.x; i < RB * CB; i += 256) tot += sens[(long)n * RB * CB + i];
  for (int off = 32; off > 0; off >>= 1) tot += __shfl_down(tot, off, 64);
  if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int total = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    int S = (2 * total + RB) / (2 * RB);
    S_s = S < CB ? S : CB;
  }
  __syncthreads();
  const int S = S_s;
  const int* cnt = count + (long)band * CB;
  const int* smp = samples + (long)band * CB;
  for (int cb = threadIdx.x; cb < CB; cb += 256) {
    uint8_t sv = sens[(long)band * CB + cb];
    if (balance) {
      // rank = number of blocks of the band that come before this one
      const long ca = cnt[cb], sa = smp[cb];
      int rank = 0;
      for (int o = 0; o < CB; ++o) {
        const long lhs = (long)cnt[o] * sa, rhs = ca * (long)smp[o];  // o before cb iff cnt_o/smp_o > cnt_cb/smp_cb
        rank += (lhs > rhs || (lhs == rhs && o < cb)) ? 1 : 0;
      }
      sv = rank < S ? 1 : 0;
    }
    if (sens_out) sens_out[(long)band * CB + cb] = sv;
    const uint32_t u = sens_draw(prefix, (uint64_t)band * (uint64_t)CB + (uint64_t)cb);
    block_keep[(long)band * CB + cb] = ((uint64_t)u < (sv ? tm : tn)) ? 0 : 1;
  }
}

static int32_t sens_geom(SensGeom& g, int32_t dtype, int N, int C, int H, int W, int kh, int kw, int stride, int pad, int x,
                         int y) {
  if (dtype != ARD_F32 && dtype != ARD_BF16) return fail(ARD_EDTYPE, "unknown dtype %d", dtype);
  if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || kh <= 0 || kw <= 0 || stride <= 0 || pad < 0)
    return fail(ARD_ESHAPE, "non-positive convolution size");
  if (H + 2 * pad < kh || W + 2 * pad < kw) return fail(ARD_ESHAPE, "kernel larger than the padded input");
  g = SensGeom{N, C, H, W, kh, kw, stride, pad, (H + 2 * pad - kh) / stride + 1, (W + 2 * pad - kw) / stride + 1, 0, 0, 0, 0, 0, 0};
  g.rows = g.Ho * g.Wo;
  if ((long)C * kh * kw > 0x7fffff00L || (long)N * g.rows > 0x7fffff00L) return fail(ARD_ESHAPE, "input matrix too large");
  g.cols = C * kh * kw;
  if (x < 1 || y < 0) return fail(ARD_EINVAL, "region size must be positive (y = 0: the whole width)");
  g.x = x;
  g.y = y == 0 ? g.cols : y;
  g.RB = ceil_div(g.rows, g.x);
  g.CB = ceil_div(g.cols, g.y);
  if ((long)N * g.RB * g.CB > 0x7fffff00L) return fail(ARD_ESHAPE, "too many regions");
  return ARD_OK;
}

}  // namespace ard

using namespace ard;

extern "C" int32_t ard_sens_regions(int32_t N, int32_t C, int32_t H, int32_t Wd, int32_t kh, int32_t kw, int32_t stride,
                                    int32_t pad, int32_t x, int32_t y, int32_t* rows, int32_t* row_bands,
                                    int32_t* col_blocks) {
  SensGeom g;
  if (int32_t st = sens_geom(g, ARD_BF16, N, C, H, Wd, kh, kw, stride, pad, x, y)) return st;
  if (rows) *rows = g.rows;
  if (row_bands) *row_bands = g.RB;
  if (col_blocks) *col_blocks = g.CB;
  return ARD_OK;
}

extern "C" int32_t ard_sens_predict(int32_t dtype, int32_t N, int32_t C, int32_t H, int32_t Wd, int32_t kh, int32_t kw,
                                    int32_t stride, int32_t pad, int32_t x, int32_t y, int32_t k_permille,
                                    int32_t t_permille, float threshold, uint64_t seed, uint64_t iteration, const void* A,
                                    int32_t* d_count, int32_t* d_samples, uint8_t* d_sens, void* stream) {
  BatchSuspend not_recorded;
  SensGeom g;
  if (int32_t st = sens_geom(g, dtype, N, C, H, Wd, kh, kw, stride, pad, x, y)) return st;
  if (k_permille < 1 || k_permille > 1000 || t_permille < 0 || t_permille > 1000)
    return fail(ARD_EINVAL, "k and t are per-mille values (k in 1..1000, t in 0..1000)");
  if ((long)g.x * g.y > (1L << 31) - 1 || ((long)k_permille * g.x * g.y) / 1000 > 65536)
    return fail(ARD_ESHAPE, "a region may hold at most 65536 samples (x * y * k / 1000)");
  if (!A || !d_count || !d_samples || !d_sens) return fail(ARD_EINVAL, "null pointer");
  const uint64_t prefix = sens_prefix(seed, iteration, SENS_STREAM_SAMPLE);
  const unsigned regions = (unsigned)((long)N * g.RB * g.CB);
  // tabulated geometry when it fits: the width of every region is g.y except the clipped last column block,
  // which only exists when the width does not divide the matrix -- then each region would need its own divisor
  const bool lut_ok = g.y <= kSensLutCols && g.x <= kSensLutRows && (long)C * H * Wd < (1L << 24) && kh < 16 && kw < 16 &&
                      (long)(g.Ho - 1) * stride < 65536 && (long)(g.Wo - 1) * stride < 32768 && g.cols % g.y == 0;
  if (lut_ok) {
    const FastDiv dw = fast_div((uint32_t)g.y);
    // footprint of a region in LDS when it fits: rows a band can touch x whole width x channels of a block
    const int taps = kh * kw;
    const int nch_max = imin(C, (g.y + taps - 2) / taps + 1);
    // Bands per workgroup.  Consecutive bands touch nearly the same input rows when they are shorter than an output row
    // (98 bands of 8 positions would copy a 28 x 28 image 14 times over), so a workgroup takes several.  The pass takes as
    // long as the CU with the most workgroups, L of them: L (1600 ns + 0.8 ns per staged word, 1.6 in fp32, + 0.24 ns per
    // draw), 0.30 for one that has the CU to itself; fitted to 29 layers (8 - 128 images, 18 - 408 channels, 7 x 7 - 56 x 56, 1 -
    // 784 bands) in up to 7 groupings each, 14 % rms.  Tried: the groupings that give every CU up to 1, 2, ... 8.  The choice is
    // within 0.3 % of the best in the mean; always a little above two for every CU was 9 % slower (35 x 41 channels of
    // 56 x 56 in bands of 4: 525 workgroups 41 us, 490 30; 59 x 128 of 56 x 56 in blocks of 112 x 576: 590 91, 472 76).
    // No grouping takes more LDS than two workgroups of a CU may have.
    const int words = (Wd + 2 * pad + 31) / 32;
    int RBG = 0, G = 1, nrow = 0;
    size_t stage_bytes = 0;
    auto group = [&](int groups) {  // sets G, nrow and stage_bytes; do they fit?
      G = ceil_div(g.RB, groups);
      // output rows a group can span: groups of whole rows start on a row, any other may start anywhere in one
      const long span = (long)G * g.x;
      const long oh_span = span % g.Wo == 0 ? span / g.Wo : (span + g.Wo - 2) / g.Wo + 1;
      nrow = ((int)(oh_span < g.Ho ? oh_span : g.Ho) - 1) * stride + kh;
      stage_bytes = ((size_t)nrow * words * nch_max + g.y + (size_t)G * g.x) * 4 + G * sizeof(SensBand);
      return stage_bytes <= (size_t)4608 * kSensWaves;
    };
    const long blocks = (long)N * g.CB;  // per group of an image's bands
    const double draws = (double)k_permille * g.x * g.y / 1000, word_ns = dtype == ARD_BF16 ? 0.8 : 1.6;
    double least = 0;
    int tried = 0;
    for (int r = 1; r <= 8; ++r) {
      const int groups = (int)imin(g.RB, imax(1, (int)(256L * r / blocks)));
      if (groups == tried) continue;
      tried = groups;
      if (!group(groups)) continue;
      const long L = (blocks * ceil_div(g.RB, G) + 255) / 256;
      const double ns = L * (1600 + word_ns * nrow * words * nch_max + (L == 1 ? 0.30 : 0.24) * G * draws);
      if (!RBG || ns < least) least = ns, RBG = groups;
    }
    if (RBG) {
      group(RBG);
    } else {
      // No more bands than this fit, counting no row that is touched in part: tried from there on, one number of bands after
      // another (a 188 x 98 layer of 910 channels in bands of one position: 18 thousand tries from the top).
      const double row_bytes = 4.0 * words * nch_max * stride, top_rows = 1.0 + (double)g.x / g.Wo;
      const double room = 4608.0 * kSensWaves - 4.0 * g.y - 4.0 * words * nch_max * kh + row_bytes * top_rows;
      const int most = (int)fmin(fmax(room / (row_bytes * g.x / g.Wo + 4.0 * g.x + sizeof(SensBand)), 1.0), (double)g.RB);
      for (RBG = tried; !group(RBG) && G > 1;) RBG = imax(ceil_div(g.RB, G - 1), ceil_div(g.RB, most));
    }
    RBG = ceil_div(g.RB, G);
    // (pad < filter size: every window then starts inside the image, which the copy's bounds rely on)
    if ((((uintptr_t)A) & 15) == 0 && stage_bytes <= 150 * 1024 && (long)nrow * words * 32 * nch_max < (1L << 30) && pad < kh && pad < kw) {
      const SensStage sg{nrow, words, fast_div((uint32_t)taps), fast_div((uint32_t)kw), fast_div((uint32_t)g.Wo), fast_div((uint32_t)words),
                         fast_div((uint32_t)(nrow * words)), G, RBG};
      const unsigned groups = (unsigned)((long)N * RBG * g.CB);
      hipError_t e = hipSuccess;
      if (dtype == ARD_BF16) {
        if (stage_bytes > 65536) e = raise_lds_limit((const void*)sens_predict_staged_kernel<uint16_t>, (int)stage_bytes);
        if (e == hipSuccess)
          ARD_LAUNCH(sens_predict_staged_kernel<uint16_t>, dim3(groups), dim3(64 * kSensWaves), stage_bytes, (hipStream_t)stream,
                     (const uint16_t*)A, g, sg, k_permille, t_permille, threshold, prefix, d_count, d_samples, d_sens);
      } else {
        if (stage_bytes > 65536) e = raise_lds_limit((const void*)sens_predict_staged_kernel<float>, (int)stage_bytes);
        if (e == hipSuccess)
          ARD_LAUNCH(sens_predict_staged_kernel<float>, dim3(groups), dim3(64 * kSensWaves), stage_bytes, (hipStream_t)stream, (const float*)A, g,
                     sg, k_permille, t_permille, threshold, prefix, d_count, d_samples, d_sens);
      }
      if (e != hipSuccess) return fail(ARD_EHIP, "raising the LDS limit failed: %s", hipGetErrorString(e));
      ARD_LAUNCH_CHECK("sens_predict_staged_kernel");
      return ARD_OK;
    }
    const size_t lds = (size_t)(g.y + g.x) * sizeof(int);
    if (dtype == ARD_BF16)
      ARD_LAUNCH(sens_predict_lut_kernel<uint16_t>, dim3(regions), dim3(256), lds, (hipStream_t)stream, (const uint16_t*)A, g, k_permille,
                 t_permille, threshold, prefix, dw, d_count, d_samples, d_sens);
    else
      ARD_LAUNCH(sens_predict_lut_kernel<float>, dim3(regions), dim3(256), lds, (hipStream_t)stream, (const float*)A, g, k_permille,
                 t_permille, threshold, prefix, dw, d_count, d_samples, d_sens);
    ARD_LAUNCH_CHECK("sens_predict_lut_kernel");
    return ARD_OK;
  }
  if (dtype == ARD_BF16)
    ARD_LAUNCH(sens_predict_kernel<uint16_t>, dim3(regions), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)A, g, k_permille,
               t_permille, threshold, prefix, d_count, d_samples, d_sens);
  else
    ARD_LAUNCH(sens_predict_kernel<float>, dim3(regions), dim3(256), 0, (hipStream_t)stream, (const float*)A, g, k_permille,
               t_permille, threshold, prefix, d_count, d_samples, d_sens);
  ARD_LAUNCH_CHECK("sens_predict_kernel");
  return ARD_OK;
}

extern "C" int32_t ard_sens_row_pattern(int32_t N, int32_t rows, int32_t x, const uint8_t* d_sens, double m, double n,
                                        uint64_t seed, uint64_t iteration, uint8_t* d_mask, int32_t* d_keep, int32_t* d_count,
                                        void* stream) {
  BatchSuspend not_recorded;
  if (N <= 0 || rows <= 0 || x <= 0) return fail(ARD_ESHAPE, "N, rows and x must be positive");
  if ((long)N * rows > 0x7fffff00L) return fail(ARD_ESHAPE, "too many rows");
  if (!(m >= 0.0 && m <= 1.0) || !(n >= 0.0 && n <= 1.0)) return fail(ARD_EINVAL, "possibilities must lie in [0, 1]");
  if (!d_sens || (!d_mask && !d_keep && !d_count)) return fail(ARD_EINVAL, "null pointer");
  const int total = N * rows;
  const int chunk = (int)align_up((size_t)ceil_div(total, 128), 1024);  // at most 128 workgroups of whole 1024-row rounds
  const dim3 grid((unsigned)ceil_div(total, chunk));
  const uint64_t tm = sens_threshold(m), tn = sens_threshold(n), pre = sens_prefix(seed, iteration, SENS_STREAM_ROWS);
  const int RB = ceil_div(rows, x);
  const bool via_mask = d_mask && (((uintptr_t)d_mask & 15) == 0);
  if (d_mask) {
    ARD_LAUNCH(sens_row_pattern_kernel, grid, dim3(1024), 0, (hipStream_t)stream, d_sens, total, rows, x, RB, 1, tm, tn, pre, chunk, 0,
               d_mask, d_keep, d_count);
    ARD_LAUNCH_CHECK("sens_row_pattern_kernel");
    if (!d_keep && !d_count) return ARD_OK;
  }
  ARD_LAUNCH(sens_row_pattern_kernel, grid, dim3(1024), 0, (hipStream_t)stream, d_sens, total, rows, x, RB, 1, tm, tn, pre, chunk,
             via_mask ? 1 : 2, d_mask, d_keep, d_count);
  ARD_LAUNCH_CHECK("sens_row_pattern_kernel");
  return ARD_OK;
}

extern "C" int32_t ard_sens_block_pattern(int32_t N, int32_t row_bands, int32_t col_blocks, const int32_t* d_count,
                                          const int32_t* d_samples, const uint8_t* d_sens, int32_t balance, double m, double n,
                                          uint64_t seed, uint64_t iteration, uint8_t* d_sens_out, uint8_t* d_block_keep,
                                          void* stream) {
  BatchSuspend not_recorded;
  if (N <= 0 || row_bands <= 0 || col_blocks <= 0) return fail(ARD_ESHAPE, "N, row_bands and col_blocks must be positive");
  if ((long)N * row_bands * col_blocks > 0x7fffff00L) return fail(ARD_ESHAPE, "too many blocks");
  if (!(m >= 0.0 && m <= 1.0) || !(n >= 0.0 && n <= 1.0)) return fail(ARD_EINVAL, "possibilities must lie in [0, 1]");
  if (!d_sens || !d_block_keep || (balance && (!d_count || !d_samples))) return fail(ARD_EINVAL, "null pointer");
  ARD_LAUNCH(sens_block_pattern_kernel, dim3((unsigned)(N * row_bands)), dim3(256), 0, (hipStream_t)stream, d_count, d_samples,
             d_sens, row_bands, col_blocks, balance, sens_threshold(m), sens_threshold(n),
             sens_prefix(seed, iteration, SENS_STREAM_BLOCKS), d_sens_out, d_block_keep);
  ARD_LAUNCH_CHECK("sens_block_pattern_kernel");
  return ARD_OK;
}
