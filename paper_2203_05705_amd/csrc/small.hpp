// Small bf16 products of a layer in the caller's own layout, in one launch.
//
// The LDS-direct kernels want operands whose rows are whole 16-byte pieces without gaps, and few tiles want their
// contraction split, so a small layer under a row pattern was three launches a product: compact copies, the product, and a
// pass that sums, spreads the result and writes the zeros, 4 us each whatever the size.  What bounds such a product is the
// launch and one or two trips to memory.  Here a workgroup makes 32 x 32 kept outputs; its four or eight wavefronts deal the
// contraction among them in slices of 32 and fetch their MFMA operands from the maps themselves, without LDS: an operand
// that runs along the contraction S contiguous 16-byte loads per 8 elements of every S-th (any alignment: the
// vector memory unit takes it), one that runs across it 2-byte loads, 16 neighbours a row.  The
// partial sums meet in LDS, and the workgroup writes all of the output that its kept rows and columns own, zeros
// included.
#pragma once
#include <type_traits>

#include "engine.hpp"
#include "fast.hpp"

namespace ard {

struct SmallArgs {
  const uint16_t *A, *B, *gate;  // gate: zero the result where it is not positive (layout of C)
  uint16_t* C;
  int lda, ldb, ldc;
  int M, N, K;
  int am_off, am_step, bn_off, bn_step;  // kept row of C -> row of A, kept column of C -> row of B
  int ka_off, ka_step, kb_off, kb_step;  // contraction -> column (row, where it runs across) of A and of B
  int full;                              // slices of 32 that the wide loads may fetch whole
  int rm_off, rm_step, rows, cn_off, cn_step, cols;  // kept row / column -> C, and C's extents
  float alpha;
  int relu, vec;
  int tiles_m, tiles_n;
};

struct __attribute__((packed, aligned(2))) SmallPiece {
  uint32_t w[4];
};

// Eight elements of a lane, contraction k0 + 8 g .. + 7, as they come from memory.  S > 0: the operand runs along the
// contraction and keeps every S-th element; S == 0: any map.  Wide loads start at the 4-byte boundary at or before the
// first element (16 bytes from an odd element on are several times slower: 77 x 3191 -> 384, every second input, 33.9 us
// against 13.7 with rows of 2880), `odd` tells which.  They read no further than the 8 S elements, where S == 1 the
// last of these is loaded by itself.
template <int S> struct SmallRaw {
  u32x4_t q[S];
  uint32_t last, odd;
};
template <> struct SmallRaw<0> {
  uint16_t h[8];
};
struct __attribute__((packed, aligned(4))) SmallQuad {
  u32x4_t q;
};

template <int S>
__device__ __forceinline__ void small_load(SmallRaw<S>& v, const uint16_t* p, long kstride, int k0) {
  if constexpr (S > 0) {
    p += (long)k0 * S;
    v.odd = (uint32_t)((uintptr_t)p >> 1) & 1u;
    const SmallQuad* q = reinterpret_cast<const SmallQuad*>((uintptr_t)p & ~(uintptr_t)3);
#pragma unroll
    for (int i = 0; i < S; ++i) v.q[i] = q[i].q;
    v.last = S == 1 ? p[7] : 0;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) v.h[j] = p[(k0 + j) * kstride];
  }
}

template <int S>
__device__ __forceinline__ bf16x8_t small_value(const SmallRaw<S>& v) {
  uint4 r;
  uint32_t* w = reinterpret_cast<uint32_t*>(&r);
  if constexpr (S > 0) {
    u32x4_t q[S];
#pragma unroll
    for (int i = 0; i < S; ++i) {
      q[i] = v.q[i];
      asm volatile("" : "+v"(q[i]));  // (else a load is narrowed to the words that are used, one each)
    }
    auto word = [&](int i) { return i < 4 * S ? q[i / 4][i % 4] : v.last; };
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      // elements j S (even) and (j + 1) S, counted from the boundary: one further where the first is odd
      const int e0 = j * S, e1 = e0 + S;
      const uint32_t lo = (word(e0 / 2) >> (16 * v.odd)) & 0xffffu;
      const uint32_t hi = (e1 & 1) ? __builtin_amdgcn_alignbit(word((e1 + 1) / 2), word(e1 / 2), 16 * v.odd) & 0xffff0000u
                                   : (word(e1 / 2) >> (16 * v.odd)) << 16;
      w[j / 2] = lo | hi;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; j += 2) w[j / 2] = (uint32_t)v.h[j] | ((uint32_t)v.h[j + 1] << 16);
  }
  return __builtin_bit_cast(bf16x8_t, r);
}

// the last slice: indices clamped, what lies beyond the contraction zero
__device__ __forceinline__ bf16x8_t small_tail(const uint16_t* p, long kstride, int k0, int K) {
  SmallRaw<0> v;
#pragma unroll
  for (int j = 0; j < 8; ++j) v.h[j] = p[min(k0 + j, K - 1) * kstride];
#pragma unroll
  for (int j = 0; j < 8; ++j) v.h[j] = k0 + j < K ? v.h[j] : (uint16_t)0;
  return small_value<0>(v);
}

// SA, SB: see SmallRaw.  A_KC, B_KC: the operand runs along the contraction.  Eight sums whatever the number of wavefronts,
// sum v of slices v, v + 8, ..: a grouped launch, whose four wavefronts make SUMS = 2 of them each, gives the very bits of a
// launch by itself.  (Four wavefronts with one sum each are right where there are no more than four slices: the
// others would be zeros.)
// lds: small_lds_bytes(sums)
constexpr int kSmallRed = 32 * 33, kSmallTile = 32 * 34;
constexpr size_t small_lds_bytes(int sums) { return (size_t)sums * kSmallRed * 4 + kSmallTile * 2; }
template <bool A_KC, bool B_KC, int SA, int SB, int SUMS>
__device__ __forceinline__ void small_body(const SmallArgs& P, const int block_id, const int threads, void* lds) {
  uint16_t* const tile = (uint16_t*)lds;
  float* const red = (float*)(tile + kSmallTile);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4;
  const int waves = threads >> 6;  // 4 or 8
  const int tm = block_id / P.tiles_n, tn = block_id - tm * P.tiles_n;
  const int m0 = tm * 32, n0 = tn * 32;
  const uint16_t *pa[2], *pb[2];
  const long ka = A_KC ? P.ka_step : (long)P.ka_step * P.lda, kb = B_KC ? P.kb_step : (long)P.kb_step * P.ldb;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    // (rows beyond the last are copies of it: their results are not stored)
    const long ra = P.am_off + (long)min(m0 + 16 * t + (lane & 15), P.M - 1) * P.am_step;
    const long rb = P.bn_off + (long)min(n0 + 16 * t + (lane & 15), P.N - 1) * P.bn_step;
    pa[t] = P.A + (A_KC ? ra * P.lda + P.ka_off : ra + (long)P.ka_off * P.lda);
    pb[t] = P.B + (B_KC ? rb * P.ldb + P.kb_off : rb + (long)P.kb_off * P.ldb);
  }
  f32x4_t acc[SUMS][2][2] = {};
  auto multiply = [&](f32x4_t (&c)[2][2], const bf16x8_t (&a)[2], const bf16x8_t (&b)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], c[i][j], 0, 0, 0);
  };
  // U slices under way at once, loads unconditional (behind branches every one would be waited for by itself)
  auto slices = [&](auto count, auto first, int s) {
    constexpr int U = decltype(count)::value, F = decltype(first)::value;
    SmallRaw<SA> va[U][2];
    SmallRaw<SB> vb[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        small_load<SA>(va[u][t], pa[t], ka, 32 * (s + u * waves) + 8 * g);
        small_load<SB>(vb[u][t], pb[t], kb, 32 * (s + u * waves) + 8 * g);
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bf16x8_t a[2] = {small_value<SA>(va[u][0]), small_value<SA>(va[u][1])};
      const bf16x8_t b[2] = {small_value<SB>(vb[u][0]), small_value<SB>(vb[u][1])};
      multiply(acc[(F + u) % SUMS], a, b);
    }
  };
  constexpr int U = SA == 1 && SB == 1 ? 4 : 2;
  int s = wave;
  for (; s + (U - 1) * waves < P.full; s += U * waves) slices(std::integral_constant<int, U>{}, std::integral_constant<int, 0>{}, s);
  if (s < P.full) slices(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{}, s);
  if (U > 2 && s + waves < P.full) slices(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, s + waves);
  if (U > 2 && s + 2 * waves < P.full) slices(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{}, s + 2 * waves);
  if (wave == P.full % waves && 32 * P.full < P.K) {
    const int k0 = 32 * P.full + 8 * g;
    const bf16x8_t a[2] = {small_tail(pa[0], ka, k0, P.K), small_tail(pa[1], ka, k0, P.K)};
    const bf16x8_t b[2] = {small_tail(pb[0], kb, k0, P.K), small_tail(pb[1], kb, k0, P.K)};
    if (SUMS == 2 && (P.full / waves) % 2) multiply(acc[SUMS - 1], a, b);
    else multiply(acc[0], a, b);
  }
#pragma unroll
  for (int v = 0; v < SUMS; ++v)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(wave + v * waves) * kSmallRed + (16 * i + 4 * g + r) * 33 + 16 * j + (lane & 15)] = acc[v][i][j][r];
  __syncthreads();
  for (int e = tid; e < 1024; e += threads) {
    const int r = e >> 5, c = e & 31;
    const float* const p = red + r * 33 + c;
    float x = (p[0] + p[kSmallRed]) + (p[2 * kSmallRed] + p[3 * kSmallRed]);
    x += waves * SUMS == 8 ? (p[4 * kSmallRed] + p[5 * kSmallRed]) + (p[6 * kSmallRed] + p[7 * kSmallRed]) : 0.0f;
    x *= P.alpha;
    if (P.relu) x = fmaxf(x, 0.0f);
    tile[r * 34 + c] = f32_to_bf16_bits(x);
  }
  __syncthreads();
  // what this tile's kept rows and columns own: groups [j * step, (j + 1) * step), the last ones up to the end
  const int r0 = m0 * P.rm_step, r1 = tm + 1 < P.tiles_m ? r0 + 32 * P.rm_step : P.rows;
  const int c0 = n0 * P.cn_step, c1 = tn + 1 < P.tiles_n ? c0 + 32 * P.cn_step : P.cols;
  const unsigned pieces = (unsigned)(c1 - c0 + 7) / 8, total = (unsigned)(r1 - r0) * pieces;
  for (unsigned i = tid; i < total; i += threads) {
    const unsigned ri = i / pieces;
    const int r = r0 + (int)ri, c = c0 + 8 * (int)(i - ri * pieces);
    const int dr = r - P.rm_off, m = dr < 0 ? 0 : (int)((unsigned)dr / (unsigned)P.rm_step);
    const long at = (long)r * P.ldc + c;
    SmallPiece v{};
    if (dr >= 0 && m * P.rm_step == dr && m < P.M) {
      const int dc = c - P.cn_off;
      int n = dc <= 0 ? 0 : (int)((unsigned)(dc + P.cn_step - 1) / (unsigned)P.cn_step);  // first kept column at or after c
      int next = P.cn_off + n * P.cn_step;
      const uint16_t* const row = tile + (m - m0) * 34 - n0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool hit = next == c + e && n < P.N && c + e < c1;
        uint32_t x = hit ? row[min(n, n0 + 31)] : 0u;
        if (hit && P.gate && !(bf16_bits_to_f32(P.gate[at + e]) > 0.0f)) x = 0u;
        v.w[e / 2] |= x << (16 * (e & 1));
        n += hit ? 1 : 0;
        next += hit ? P.cn_step : 0;
      }
    }
    if (c + 8 <= c1) {
      if (P.vec) *reinterpret_cast<uint4*>(P.C + at) = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]);
      else *reinterpret_cast<SmallPiece*>(P.C + at) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 7; ++e)
        if (c + e < c1) P.C[at + e] = (uint16_t)(v.w[e / 2] >> (16 * (e & 1)));
    }
  }
}

// The forms there are, by kind.  KK + S: both operands run along the contraction and keep every S-th element, K1 + S: A is
// compact; KM + S: B runs across it (data gradients); MM: both do (weight gradients).  S = 0: any other step.
enum { GK_SMALL_KK = 110, GK_SMALL_K1 = 115, GK_SMALL_KM = 120, GK_SMALL_MM = 125 };
static inline bool small_kind(int kind) { return kind >= GK_SMALL_KK && kind <= GK_SMALL_MM; }
template <bool A_KC, bool B_KC, int SA, int SB> struct SmallForm {
  static constexpr bool a_kc = A_KC, b_kc = B_KC;
  static constexpr int sa = SA, sb = SB;
};
// what a grouped launch holds: products of compact activations and weight gradients.  false: not among them
template <class F> __host__ __device__ __forceinline__ bool small_recorded(int kind, const F& f) {
  switch (kind) {
    case GK_SMALL_K1 + 0: f(SmallForm<true, true, 1, 0>{}); return true;
    case GK_SMALL_K1 + 1: f(SmallForm<true, true, 1, 1>{}); return true;
    case GK_SMALL_K1 + 2: f(SmallForm<true, true, 1, 2>{}); return true;
    case GK_SMALL_K1 + 3: f(SmallForm<true, true, 1, 3>{}); return true;
    case GK_SMALL_K1 + 4: f(SmallForm<true, true, 1, 4>{}); return true;
    case GK_SMALL_KM + 1: f(SmallForm<true, false, 1, 0>{}); return true;
    case GK_SMALL_MM: f(SmallForm<false, false, 0, 0>{}); return true;
    default: return false;
  }
}
bool batch_push_small(int kind, const SmallArgs& a, int gx);
// (small.hip)
void launch_small_alone(int kind, const SmallArgs& P, unsigned tiles, unsigned threads, hipStream_t stream);

}  // namespace ard
