// One time step of the fp32 recurrences in one launch: the recurrent product of 16 batch rows x 16 kept units and the cell
// that takes it.  As two launches (product, cell) a step cost two fixed costs of 4 us and a trip of the product's result
// through memory, which is what bounds layers of this size
// (8 steps, 45 rows, 56 kept units: forward 76 -> 42 us, backward 80 -> 50; 104 rows, 384 kept units: 104 -> 71, 142 -> 108).
// Eight wavefronts deal the contraction in slices of 16, operands straight from memory to registers (a lane's 16 bytes are
// the contraction indices 4 g .. 4 g + 3 of the four 16x16x4 MFMAs of a slice), the sums meet in LDS in a fixed order.
#pragma once
#include "engine.hpp"

namespace ard {

constexpr int kStepWaves = 8;

struct LstmStep32 {
  const float *whc;              // [4Hp x Hp]
  const float *G, *hc_prev;      // fwd: [B x 4Hp] input projections; [B x Hp] (NULL: first step)
  const float *c_prev;           // [B x H] (NULL: first step)
  float *gates, *c, *h, *hc;     // fwd: results [B x 4H], [B x H], [B x H], [B x Hp]; bwd: gates and c are read
  const float *dh, *dG_next;     // bwd: [B x H]; [B x 4Hp] (NULL: last step)
  float *dc, *dG;                // bwd: [B x H] carried from step to step; [B x 4Hp]
  int B, H, Hk, Hp, off, step;   // kept unit j is unit off + j * step
};

__global__ __launch_bounds__(64 * kStepWaves) void lstm_step32_fwd_kernel(const LstmStep32 P) {
  __shared__ float red[kStepWaves][4][16 * 17];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4;
  const int j0 = blockIdx.x * 16, b0 = blockIdx.y * 16, Hp = P.Hp;
  // the cell's own operands are under way during the product (256 threads: row tid / 16, unit tid % 16)
  const int b = b0 + (tid >> 4), j = j0 + (tid & 15), u = P.off + j * P.step;
  const bool mine = tid < 256 && b < P.B && j < Hp, live = mine && j < P.Hk;
  float z[4] = {0.0f, 0.0f, 0.0f, 0.0f}, cp = 0.0f;
  if (live) {
#pragma unroll
    for (int q = 0; q < 4; ++q) z[q] = P.G[(long)b * 4 * Hp + q * Hp + j];
    if (P.c_prev) cp = P.c_prev[(long)b * P.H + u];
  }
  if (P.hc_prev) {
    // (rows beyond the last are copies of it: their results are not stored)
    const float* const pa = P.hc_prev + (long)min(b0 + (lane & 15), P.B - 1) * Hp + 4 * g;
    const float* const pb = P.whc + (long)min(j0 + (lane & 15), Hp - 1) * Hp + 4 * g;
    f32x4_t acc[4] = {};
    auto slices = [&](auto count, int s) {
      constexpr int U = decltype(count)::value;
      f32x4_t a[U], w[U][4];
#pragma unroll
      for (int v = 0; v < U; ++v) {
        a[v] = *reinterpret_cast<const f32x4_t*>(pa + 16 * (s + v * kStepWaves));
#pragma unroll
        for (int q = 0; q < 4; ++q) w[v][q] = *reinterpret_cast<const f32x4_t*>(pb + (long)q * Hp * Hp + 16 * (s + v * kStepWaves));
      }
#pragma unroll
      for (int v = 0; v < U; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][e], w[v][q][e], acc[q], 0, 0, 0);
    };
    const int full = Hp / 16;
    int s = wave;
    for (; s + 3 * kStepWaves < full; s += 4 * kStepWaves) slices(std::integral_constant<int, 4>{}, s);
    for (; s < full; s += kStepWaves) slices(std::integral_constant<int, 1>{}, s);
    if ((Hp & 8) && wave == full % kStepWaves) {  // half a slice: the upper lanes read the last one's indices again and add zeros
      const int back = g < 2 ? 16 * full : 16 * full - 8;
      const f32x4_t a = *reinterpret_cast<const f32x4_t*>(pa + back);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4_t w = *reinterpret_cast<const f32x4_t*>(pb + (long)q * Hp * Hp + back);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(g < 2 ? a[e] : 0.0f, g < 2 ? w[e] : 0.0f, acc[q], 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][q][(4 * g + r) * 17 + (lane & 15)] = acc[q][r];
    __syncthreads();
    if (live)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kStepWaves; ++w) t += red[w][q][(tid >> 4) * 17 + (tid & 15)];
        z[q] += t;
      }
  }
  if (!mine) return;
  if (!live) {
    P.hc[(long)b * Hp + j] = 0.0f;
    return;
  }
  const float gi = sigmoidf_(z[0]), gf = sigmoidf_(z[1]), gg = tanhf(z[2]), go = sigmoidf_(z[3]);
  const float cv = gf * cp + gi * gg, hv = go * tanhf(cv);
  P.hc[(long)b * Hp + j] = hv;
  // the kept unit and the zeros of the dropped ones of its group [j * step, (j + 1) * step), the last one's up to the end
  const int u1 = j + 1 < P.Hk ? (j + 1) * P.step : P.H;
  float* const ga = P.gates + (long)b * 4 * P.H;
  for (int v = j * P.step; v < u1; ++v) {
    const bool kept = v == u;
    ga[v] = kept ? gi : 0.0f, ga[P.H + v] = kept ? gf : 0.0f, ga[2 * P.H + v] = kept ? gg : 0.0f, ga[3 * P.H + v] = kept ? go : 0.0f;
    P.c[(long)b * P.H + v] = kept ? cv : 0.0f;
    P.h[(long)b * P.H + v] = kept ? hv : 0.0f;
  }
}

__global__ __launch_bounds__(64 * kStepWaves) void lstm_step32_bwd_kernel(const LstmStep32 P) {
  __shared__ float red[kStepWaves][16 * 17];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4;
  const int j0 = blockIdx.x * 16, b0 = blockIdx.y * 16, Hp = P.Hp;
  const int b = b0 + (tid >> 4), j = j0 + (tid & 15), u = P.off + j * P.step;
  const bool mine = tid < 256 && b < P.B && j < Hp, live = mine && j < P.Hk;
  float gi = 0, gf = 0, gg = 0, go = 0, cv = 0, cp = 0, dh = 0, dc = 0;
  if (live) {
    const float* const ga = P.gates + (long)b * 4 * P.H;
    const long at = (long)b * P.H + u;
    gi = ga[u], gf = ga[P.H + u], gg = ga[2 * P.H + u], go = ga[3 * P.H + u];
    cv = P.c[at], dh = P.dh[at];
    if (P.c_prev) cp = P.c_prev[at];
    if (P.dG_next) dc = P.dc[at];
  }
  if (P.dG_next) {
    const float* const pa = P.dG_next + (long)min(b0 + (lane & 15), P.B - 1) * 4 * Hp + 4 * g;
    const float* const pb = P.whc + (long)(4 * g) * Hp + min(j0 + (lane & 15), Hp - 1);
    f32x4_t acc = {};
    auto slices = [&](auto count, int s) {
      constexpr int U = decltype(count)::value;
      f32x4_t a[U];
      float w[U][4];
#pragma unroll
      for (int v = 0; v < U; ++v) {
        a[v] = *reinterpret_cast<const f32x4_t*>(pa + 16 * (s + v * kStepWaves));
#pragma unroll
        for (int e = 0; e < 4; ++e) w[v][e] = pb[(long)(16 * (s + v * kStepWaves) + e) * Hp];
      }
#pragma unroll
      for (int v = 0; v < U; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][e], w[v][e], acc, 0, 0, 0);
    };
    const int full = Hp / 4;  // (4Hp is a multiple of 32)
    int s = wave;
    for (; s + 7 * kStepWaves < full; s += 8 * kStepWaves) slices(std::integral_constant<int, 8>{}, s);
    for (; s + kStepWaves < full; s += 2 * kStepWaves) slices(std::integral_constant<int, 2>{}, s);
    if (s < full) slices(std::integral_constant<int, 1>{}, s);
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][(4 * g + r) * 17 + (lane & 15)] = acc[r];
    __syncthreads();
    if (live) {
      float t = 0.0f;
#pragma unroll
      for (int w = 0; w < kStepWaves; ++w) t += red[w][(tid >> 4) * 17 + (tid & 15)];
      dh += t;
    }
  }
  if (!mine) return;
  float* const d = P.dG + (long)b * 4 * Hp + j;
  if (!live) {
    d[0] = d[Hp] = d[2 * Hp] = d[3 * Hp] = 0.0f;
    return;
  }
  const float tc = tanhf(cv);
  dc = dh * go * (1.0f - tc * tc) + dc;
  d[0] = dc * gg * gi * (1.0f - gi);
  d[Hp] = dc * cp * gf * (1.0f - gf);
  d[2 * Hp] = dc * gi * (1.0f - gg * gg);
  d[3 * Hp] = dh * tc * go * (1.0f - go);
  P.dc[(long)b * P.H + u] = dc * gf;
}

}  // namespace ard
