// Kernels of the block-based sensitivity-aware pattern (Section 5.2.2), bf16, stride 1, on tiles of 64 channels x 128 positions:
// the forward pass, blocks of whole 64-channel groups by bands of any number of positions, and the data gradient, blocks of
// whole 64-channel groups by bands of whole output rows, filters that keep the image's size.
//
// Forward: Y[row, p] = sum over the kept blocks of p's band.  Where bands are long enough to be column tiles of their own, the
// LDS-direct product takes lists of kept steps (BlockPlan); here a tile is 128 positions wherever the bands end: it leaves
// out the channel groups that none of its positions keeps, and where a group is kept for some, the lanes of the others
// load zeros.
// Data gradient: dA[channels of group cb] = W^T * dY with the positions of cb's dropped bands taken as zero.  One launch covers
// all groups from ONE unmasked copy of dY: a workgroup takes 64 channels of a group and a run of positions (bands, or parts
// of one), leaves out the filter rows whose source rows are all dropped for its group, and where a filter row reads
// kept and dropped bands, the lanes of the dropped pixels load zeros.  (What the kept positions alone would cost, and when
// that is less: conv_scatter.hpp.)
//
// Every wavefront computes the whole 64 x 128 tile over its own quarter (16) of each 64-deep step: six LDS reads for eight
// MFMAs where 64 x 32 tiles side by side would need three for two, and one barrier a step; the four accumulators meet in LDS
// at the end.  What is left to bound it is the path from L2 into LDS (24 KB per step of 256 MFMA clocks).
// Forward, before, on the general engine's patch loaders, whole training steps, us: 37 images of 256 channels of 28 x 28 -> 247,
// bands of two rows 1837 -> 179; 8 of 448 channels of 32 x 32 -> 24, four rows 1402 -> 91; 16 of 64 channels of 14 x 14 -> 16
// 255 -> 55.  Data gradient, before, as a masked pass per column block: 128 x 256 channels of 28 x 28 -> 256, bands of 4 rows
// x 64 channels, 30 % kept: 4 x (copy 23 + product 60) us -> copy 28 + product 131.
//
// Results: positions that a tile takes along although their block is dropped multiply its weights by zeros, which a weight that is
// not finite makes NaN.  Such a result is summed again over what it consists of.  (No finite sum had such a term: two comparisons
// for every four results are all that is paid for it.)
#pragma once
#include "fast.hpp"

namespace ard {

constexpr int kBlockStages = 3, kBlockLds = kBlockStages * (64 + 128) * 128, kBlockPitch = 136;  // (positions of a row of the result; rows 272 bytes apart)

// load_stage(s, buf): step s of S into buffer buf, LDS-direct: wavefront's rows of the 64 x 64 weights, then of the 128 x 64 pixels.
template <class Load>
__device__ __forceinline__ void block_product(uint4* const lds, const int S, const int lane, const int wave, const Load& load_stage, f32x16_t (&acc)[2][4]) {
  constexpr int NST = kBlockStages, OPA = 64 * LDS_ROW_U4, OPB = 128 * LDS_ROW_U4;
#pragma unroll
  for (int im = 0; im < 2; ++im)
#pragma unroll
    for (int in = 0; in < 4; ++in)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[im][in][v] = 0.0f;
  if (S == 0) return;
  const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)lds);
  unsigned aaddr[2], baddr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = i * 32 + (lane & 31), xr = kc_swz<true>(row);
    const unsigned at = (unsigned)(row * 8 + ((2 * wave + (lane >> 5)) ^ xr)) * 16u;
    if (i < 2) aaddr[i & 1] = lds_base + at;
    baddr[i] = lds_base + (unsigned)(NST * OPA) * 16u + at;
  }
  Frag fa[2][2], fb[2][4];
  auto issue = [&](auto bufc, int set) {
    constexpr int BUF = decltype(bufc)::value;
#pragma unroll
    for (int i = 0; i < 2; ++i) lds_read_b128<BUF * OPA * 16>(fa[set][i].v, aaddr[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds_read_b128<BUF * OPB * 16>(fb[set][i].v, baddr[i]);
  };
  constexpr int LPS = 2 + DirectLoader<true, 128, 4, true>::NI;
  auto step = [&](auto bufc, auto setc, int it) {
    constexpr int BUF = decltype(bufc)::value, SET = decltype(setc)::value;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < 2; ++i) frag_wait<true>(fa[SET][i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) frag_wait<true>(fb[SET][i]);
    if (it + 1 < S) {
      if (it + NST - 1 < S) wait_vmcnt<(NST - 2) * LPS>();
      else wait_vmcnt<0>();
      wg_barrier();  // stage it+1 is complete, and every wavefront holds its part of stage it in registers
      issue(std::integral_constant<int, (BUF + 1) % NST>{}, SET ^ 1);
    }
#pragma unroll
    for (int im = 0; im < 2; ++im)
#pragma unroll
      for (int in = 0; in < 4; ++in)
        acc[im][in] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_value<true>(fa[SET][im]), frag_value<true>(fb[SET][in]), acc[im][in], 0, 0, 0);
    if (it + NST < S) load_stage(it + NST, BUF);
  };
#pragma unroll
  for (int st = 0; st < NST; ++st)
    if (st < S) load_stage(st, st);
  if (S >= NST) wait_vmcnt<(NST - 1) * LPS>();
  else wait_vmcnt<0>();
  wg_barrier();
  issue(std::integral_constant<int, 0>{}, 0);
  for (int it = 0; it < S; it += 2 * NST)
    static_for<2 * NST>([&](auto b) {
      constexpr int B = decltype(b)::value;
      if (it + B < S) step(std::integral_constant<int, B % NST>{}, std::integral_constant<int, B & 1>{}, it + B);
    });
}

// Sum of the four wavefronts' tiles, 32 rows at a time: wavefront w keeps columns 32w .. 32w + 31.
// Then the tile as bf16 [64 rows][128 positions] in LDS, from where whole runs of a channel plane leave.
// again(row, col): the sum of one result over what it consists of, asked for NaN ones only.
template <class Again>
__device__ __forceinline__ void block_results(uint4* const lds, const int lane, const int wave, f32x16_t (&acc)[2][4], const Again& again) {
  float4* const sum = reinterpret_cast<float4*>(lds);  // [wave][column tile][quarter][lane]
  uint32_t words[2][8];
  bool nan = false;
#pragma unroll
  for (int im = 0; im < 2; ++im) {
    __syncthreads();
#pragma unroll
    for (int in = 0; in < 4; ++in)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        sum[((wave * 4 + in) * 4 + q) * 64 + lane] = make_float4(acc[im][in][4 * q], acc[im][in][4 * q + 1], acc[im][in][4 * q + 2], acc[im][in][4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float4 x = sum[(wave * 4 + q) * 64 + lane];  // (wavefront 0's)
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        const float4 y = sum[((w * 4 + wave) * 4 + q) * 64 + lane];
        x.x += y.x, x.y += y.y, x.z += y.z, x.w += y.w;
      }
      words[im][2 * q] = pack_bf16x2(x.x, x.y), words[im][2 * q + 1] = pack_bf16x2(x.z, x.w);
      nan |= __builtin_isunordered(x.x, x.y) | __builtin_isunordered(x.z, x.w);
    }
  }
  __syncthreads();
  uint16_t* const tile = reinterpret_cast<uint16_t*>(lds);
#pragma unroll
  for (int im = 0; im < 2; ++im)
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const int row = im * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), col = wave * 32 + (lane & 31);
      tile[row * kBlockPitch + col] = (uint16_t)words[im][v >> 1];
      tile[(row + 1) * kBlockPitch + col] = (uint16_t)(words[im][v >> 1] >> 16);
    }
  if (nan) {
    const int col = wave * 32 + (lane & 31);
#pragma unroll 1
    for (int i = 0; i < 32; ++i) {
      const int row = (i >> 4) * 32 + 8 * ((i >> 2) & 3) + 4 * (lane >> 5) + (i & 3);
      if ((tile[row * kBlockPitch + col] & 0x7fff) > 0x7f80) tile[row * kBlockPitch + col] = f32_to_bf16_bits(again(row, col));
    }
  }
  __syncthreads();
}

// Adds the products of 64 channels of one pixel and one tap
__device__ __forceinline__ float block_dot(float x, const uint16_t* w, const uint16_t* pixel) {
#pragma unroll 1
  for (int c = 0; c < 64; ++c) x += bf16_bits_to_f32(w[c]) * bf16_bits_to_f32(pixel[c]);
  return x;
}

struct BlockFwdParams {
  const uint16_t* W;     // packed weights [Cout][taps * Cp]
  const uint16_t* grid;  // A, bordered
  uint16_t* Y;
  const uint8_t* blk;
  int ldw, Cp, CG, kh, kw;
  int HW, W_, Cout, npix, HgWg, Wg;   // output plane and its width, output channels, output positions of all images
  int RB, CB, x, cg_per_blk;          // row bands of x positions, column blocks of cg_per_blk groups of 64 channels
  int mt, total, width;               // tiles of 64 output channels, workgroups, bytes per store (2, 4, 8, 16)
  FastDiv by_mt, by_hw, by_w, by_x;   // mt, HW, W_, x
};

static __global__ __launch_bounds__(256, 2) void conv_block_fwd_kernel(const BlockFwdParams P) {
  extern __shared__ uint4 bf_lds[];
  __shared__ unsigned any_s[4], all_s[4];
  constexpr int NST = kBlockStages, OPA = 64 * LDS_ROW_U4, OPB = 128 * LDS_ROW_U4;
  uint4* const lds = bf_lds;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  touch_args<(int)(sizeof(BlockFwdParams) / 64)>(P);
  // XCD x takes the x-th eighth of the tiles; the channels of a tile of positions follow each other and share its pixels in L2
  const int xcd = (int)blockIdx.x & 7, lo = (int)((long)xcd * P.total / 8), hi = (int)((long)(xcd + 1) * P.total / 8);
  const int L = lo + ((int)blockIdx.x >> 3);
  if (L >= hi) return;
  const int T = (int)fdiv((uint32_t)L, P.by_mt), row0 = (L - T * P.mt) * 64, j0 = T * 128;
  // the positions this lane fetches, and their kept channel groups (one bit each)
  constexpr int NB = DirectLoader<true, 128, 4, true>::NI;
  uint32_t voff[NB];
  unsigned kept[NB], any = 0, all = ~0u;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int q = imin(j0 + (wave * NB + j) * 8 + (lane >> 3), P.npix - 1);
    const int n = (int)fdiv((uint32_t)q, P.by_hw), p = q - n * P.HW, h = (int)fdiv((uint32_t)p, P.by_w), w = p - h * P.W_;
    voff[j] = (uint32_t)((n * P.HgWg + h * P.Wg + w) * P.Cp + DirectLoader<true, 128, 4, true>::chunk_k(lane, wave, j)) * 2u;
    const uint8_t* const m = P.blk + ((long)n * P.RB + (int)fdiv((uint32_t)p, P.by_x)) * P.CB;
    kept[j] = 0;
    for (int cb = 0; cb < P.CB; ++cb)
      if (m[cb]) kept[j] |= (unsigned)((1ull << P.cg_per_blk) - 1) << (cb * P.cg_per_blk);
    any |= kept[j], all &= kept[j];
  }
  for (int o = 8; o < 64; o <<= 1) any |= __shfl_xor(any, o, 64), all &= __shfl_xor(all, o, 64);
  if (lane == 0) any_s[wave] = any, all_s[wave] = all;
  __syncthreads();
  const unsigned groups = P.CG < 32 ? (1u << P.CG) - 1u : ~0u;
  const unsigned need = (unsigned)__builtin_amdgcn_readfirstlane((int)(any_s[0] | any_s[1] | any_s[2] | any_s[3])) & groups;
  const unsigned mixed = need & ~(unsigned)__builtin_amdgcn_readfirstlane((int)(all_s[0] & all_s[1] & all_s[2] & all_s[3]));
  const int taps = P.kh * P.kw, S = __builtin_popcount(need) * taps;
  f32x16_t acc[2][4];
  // step s = (kept channel group, tap); lane l keeps steps l and 64 + l
  auto entry = [&](int s) {
    const int i = s / taps, t = s - i * taps, r = t / P.kw;
    unsigned m = need;
    for (int k = i; k > 0; --k) m &= m - 1;
    return r | ((t - r * P.kw) << 4) | (__builtin_ctz(m | 0x80000000u) << 8);
  };
  const int e0 = entry(imin(lane, S - 1)), e1 = entry(imin(64 + lane, S - 1));
  DirectLoader<true, 64, 4, true> la;
  la.init(P.W, P.ldw, axis_identity(P.Cout), row0, lane, wave);
  const char* const gridb = reinterpret_cast<const char*>(P.grid);
  auto load_stage = [&](int s, int buf) {
    const int e = s < 64 ? __builtin_amdgcn_readlane(e0, s) : __builtin_amdgcn_readlane(e1, s - 64);
    const int r = e & 15, col = (e >> 4) & 15, cg = e >> 8;
    la.issue(lds + buf * OPA, (r * P.kw + col) * P.Cp + cg * 64, wave);
    const char* sb = gridb + (long)((r * P.Wg + col) * P.Cp + cg * 64) * 2;
    uint4* const dst = lds + NST * OPA + buf * OPB + wave * NB * 64;
    if (mixed >> cg & 1) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const char* src = kept[j] >> cg & 1 ? sb + voff[j] : reinterpret_cast<const char*>(g_zero_chunk);
        __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(src), ARD_LDS_PTR(dst + j * 64), 16, 0, 0);
      }
    } else {
#pragma unroll
      for (int j = 0; j < NB; ++j) __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(sb + voff[j]), ARD_LDS_PTR(dst + j * 64), 16, 0, 0);
    }
  };
  block_product(lds, S, lane, wave, load_stage, acc);
  block_results(lds, lane, wave, acc, [&](int row, int col) {
    const int q = imin(j0 + col, P.npix - 1);
    const int n = (int)fdiv((uint32_t)q, P.by_hw), p = q - n * P.HW, h = (int)fdiv((uint32_t)p, P.by_w), w = p - h * P.W_;
    const uint8_t* const m = P.blk + ((long)n * P.RB + (int)fdiv((uint32_t)p, P.by_x)) * P.CB;
    const uint16_t* const at = P.grid + ((long)n * P.HgWg + h * P.Wg + w) * P.Cp;
    const uint16_t* const wr = P.W + (long)imin(row0 + row, P.Cout - 1) * P.ldw;
    float x = 0.0f;
#pragma unroll 1
    for (int cg = 0; cg < P.CG && x == x; ++cg)
      if (m[cg / P.cg_per_blk])
#pragma unroll 1
        for (int t = 0; t < taps; ++t) {
          const int r = t / P.kw, s = t - r * P.kw;
          x = block_dot(x, wr + t * P.Cp + cg * 64, at + (long)(r * P.Wg + s) * P.Cp + cg * 64);
        }
    return x;
  });
  const uint16_t* const tile = reinterpret_cast<const uint16_t*>(lds);
  // a thread takes E positions of a row: they lie in one plane (host: the planes are whole pieces)
  auto store = [&](auto unit) {
    using U = decltype(unit);
    constexpr int E = (int)sizeof(U) / 2, PR = 128 / E;  // positions per store, threads per row
    const int c = (tid % PR) * E, q = j0 + c;
    if (q >= P.npix) return;
    const int n = (int)fdiv((uint32_t)q, P.by_hw), p = q - n * P.HW;
    uint16_t* const out = P.Y + ((long)n * P.Cout + row0) * P.HW + p;
    for (int r = tid / PR; r < 64 && row0 + r < P.Cout; r += 256 / PR) *reinterpret_cast<U*>(out + (long)r * P.HW) = *reinterpret_cast<const U*>(tile + r * kBlockPitch + c);
  };
  if (P.width == 16) store(uint4{});
  else if (P.width == 8) store(uint2{});
  else if (P.width == 4) store(uint32_t{});
  else store(uint16_t{});
}

struct BlockDataParams {
  const uint16_t* W;     // packed weights [C][taps * Cp], taps reversed
  const uint16_t* grid;  // dY, bordered by kh-1-pad
  uint16_t* dA;
  const uint8_t* blk;
  int ldw, Cp, CG, kh, kw, ph, pw;   // ph, pw: rows and columns of border before dY
  int H, W_, C, HgWg, Wg;
  int RB, CB, x, rows_per_band;      // bands of whole rows
  int cpb, mt;                       // channels per group, 64-row tiles per group
  int bands_per_tile, parts;         // a tile is bands_per_tile bands (parts = 1) or one of `parts` parts of a band
  int tiles_img, total, width;       // tiles per image, workgroups, bytes per store (2, 4, 16)
  FastDiv by_groups, by_tiles, by_w;  // CB * mt, tiles_img, W_
};

static __global__ __launch_bounds__(256, 2) void conv_block_data_kernel(const BlockDataParams P) {
  extern __shared__ uint4 bd_lds[];
  constexpr int NST = kBlockStages, OPA = 64 * LDS_ROW_U4, OPB = 128 * LDS_ROW_U4;
  uint4* const lds = bd_lds;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  touch_args<(int)(sizeof(BlockDataParams) / 64)>(P);
  // XCD x takes the x-th eighth of the tiles; the groups of a tile follow each other and share its pixels in L2
  const int xcd = (int)blockIdx.x & 7, lo = (int)((long)xcd * P.total / 8), hi = (int)((long)(xcd + 1) * P.total / 8);
  const int L = lo + ((int)blockIdx.x >> 3);
  if (L >= hi) return;
  const int T = (int)fdiv((uint32_t)L, P.by_groups), gm = L - T * P.CB * P.mt;
  const int n = (int)fdiv((uint32_t)T, P.by_tiles), t = T - n * P.tiles_img;
  const int cb = gm / P.mt, row0 = cb * P.cpb + (gm - cb * P.mt) * 64;
  const int HW = P.H * P.W_;
  int p0, p1;
  if (P.parts == 1) {
    p0 = t * P.bands_per_tile * P.x, p1 = imin(p0 + P.bands_per_tile * P.x, HW);
  } else {
    const int b = t / P.parts, i = t - b * P.parts;
    p0 = b * P.x + i * 128, p1 = imin(imin(p0 + 128, (b + 1) * P.x), HW);
    if (p0 >= p1) return;
  }
  // kept bands of this image and group, one bit each
  const unsigned long long bands = __ballot(lane < P.RB && P.blk[((long)n * P.RB + imin(lane, P.RB - 1)) * P.CB + cb] != 0);
  const int h_lo = p0 / P.W_, h_hi = (p1 - 1) / P.W_;
  unsigned need = 0, mixed = 0;  // filter rows with a kept source row in this tile / with a dropped one as well
  int nr = 0;
  for (int r = 0; r < P.kh; ++r) {
    const int a = imax(h_lo + r - P.ph, 0), b = imin(h_hi + r - P.ph, P.H - 1);
    if (a > b) continue;
    const int ba = a / P.rows_per_band, bb = b / P.rows_per_band;
    const unsigned long long span = (~0ull >> (63 - (bb - ba))) << ba;
    if (!(bands & span)) continue;
    need |= 1u << r;
    ++nr;
    if ((bands & span) != span) mixed |= 1u << r;
  }
  const int per_cg = imax(nr * P.kw, 1), S = nr * P.kw * P.CG;
  f32x16_t acc[2][4];
  // step s = (channel group, filter row among the needed ones, filter column); lane l keeps steps l and 64 + l
  auto entry = [&](int s) {
    const int cg = s / per_cg, i = s - cg * per_cg;
    int k = i / P.kw;
    const int col = i - k * P.kw;
    unsigned m = need;
    for (; k > 0; --k) m &= m - 1;
    return (__builtin_ctz(m | 0x80000000u) & 15) | (col << 4) | (cg << 8);
  };
  const int e0 = entry(imin(lane, S - 1)), e1 = entry(imin(64 + lane, S - 1));
  DirectLoader<true, 64, 4, true> la;
  la.init(P.W, P.ldw, axis_identity(P.C), row0, lane, wave);
  constexpr int NB = DirectLoader<true, 128, 4, true>::NI;
  uint32_t voff[NB];
  unsigned kept[NB];  // filter rows whose source pixel counts, per chunk of this lane
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int p = imin(p0 + (wave * NB + j) * 8 + (lane >> 3), p1 - 1);
    const int h = (int)fdiv((uint32_t)p, P.by_w), w = p - h * P.W_;
    voff[j] = (uint32_t)((n * P.HgWg + h * P.Wg + w) * P.Cp + DirectLoader<true, 128, 4, true>::chunk_k(lane, wave, j)) * 2u;
    kept[j] = 0;
    for (int r = 0; r < P.kh; ++r) {
      const int hs = imin(imax(h + r - P.ph, 0), P.H - 1);  // (rows outside the image are zeros in the grid already)
      kept[j] |= (unsigned)(bands >> (hs / P.rows_per_band) & 1) << r;
    }
  }
  const char* const gridb = reinterpret_cast<const char*>(P.grid);
  auto load_stage = [&](int s, int buf) {
    const int e = s < 64 ? __builtin_amdgcn_readlane(e0, s) : __builtin_amdgcn_readlane(e1, s - 64);
    const int r = e & 15, col = (e >> 4) & 15, cg = e >> 8;
    la.issue(lds + buf * OPA, (r * P.kw + col) * P.Cp + cg * 64, wave);
    const char* sb = gridb + (long)((r * P.Wg + col) * P.Cp + cg * 64) * 2;
    uint4* const dst = lds + NST * OPA + buf * OPB + wave * NB * 64;
    if (mixed >> r & 1) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const char* src = kept[j] >> r & 1 ? sb + voff[j] : reinterpret_cast<const char*>(g_zero_chunk);
        __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(src), ARD_LDS_PTR(dst + j * 64), 16, 0, 0);
      }
    } else {
#pragma unroll
      for (int j = 0; j < NB; ++j) __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(sb + voff[j]), ARD_LDS_PTR(dst + j * 64), 16, 0, 0);
    }
  };
  block_product(lds, S, lane, wave, load_stage, acc);
  block_results(lds, lane, wave, acc, [&](int row, int col) {
    const int p = imin(p0 + col, p1 - 1), h = (int)fdiv((uint32_t)p, P.by_w), w = p - h * P.W_;
    const uint16_t* const wr = P.W + (long)(row0 + row) * P.ldw;
    float x = 0.0f;
#pragma unroll 1
    for (int r = 0; r < P.kh; ++r) {
      const int hs = h + r - P.ph;
      if (hs < 0 || hs >= P.H || !(bands >> (hs / P.rows_per_band) & 1)) continue;
#pragma unroll 1
      for (int s = imax(P.pw - w, 0); s < imin(P.kw, P.W_ + P.pw - w); ++s)
#pragma unroll 1
        for (int c = 0; c < P.Cp && x == x; c += 64)
          x = block_dot(x, wr + (r * P.kw + s) * P.Cp + c, P.grid + ((long)n * P.HgWg + (h + r) * P.Wg + w + s) * P.Cp + c);
    }
    return x;
  });
  const uint16_t* const tile = reinterpret_cast<const uint16_t*>(lds);
  uint16_t* const out = P.dA + ((long)n * P.C + row0) * HW + p0;
  const int len = p1 - p0;
  auto store = [&](auto unit) {
    using U = decltype(unit);
    constexpr int E = (int)sizeof(U) / 2, PR = 128 / E;  // positions per store, threads per row
    const int c = (tid % PR) * E;
    if (c >= len) return;
    for (int r = tid / PR; r < 64; r += 256 / PR) *reinterpret_cast<U*>(out + (long)r * HW + c) = *reinterpret_cast<const U*>(tile + r * kBlockPitch + c);
  };
  if (P.width == 16) store(uint4{});
  else if (P.width == 4) store(uint32_t{});
  else store(uint16_t{});
}

// (conv_kept.hip)
int32_t launch_conv_block_fwd(const BlockFwdParams& P, hipStream_t stream);
int32_t launch_conv_block_data(const BlockDataParams& P, hipStream_t stream);

}  // namespace ard
