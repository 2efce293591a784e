// Forward pass of a convolution under the block-based sensitivity-aware pattern (Section 5.2.2), bf16, stride 1, blocks of
// whole 64-channel groups by bands of any number of positions.
//
// Y[row, p] = sum over the kept blocks of p's band.  Where bands are long enough to be column tiles of their own, the
// LDS-direct product takes lists of kept steps (BlockPlan); here a tile is 128 positions wherever the bands end: it leaves
// out the channel groups that none of its positions keeps, and where a group is kept for some, the lanes of the others
// load zeros.
//
// Every wavefront computes the whole 64 x 128 tile over its own quarter (16) of each 64-deep step: six LDS reads for eight
// MFMAs where 64 x 32 tiles side by side would need three for two, and one barrier a step; the four accumulators meet in LDS
// at the end.  What is left to bound it is the path from L2 into LDS (24 KB per step of 256 MFMA clocks).
// Before, on the general engine's patch loaders, whole training steps, us: 37 images of 256 channels of 28 x 28 -> 247, bands of
// two rows 1837 -> 179; 8 of 448 channels of 32 x 32 -> 24, four rows 1402 -> 91; 16 of 64 channels of 14 x 14 -> 16 255 -> 55.
#pragma once
#include "fast.hpp"

namespace ard {

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

constexpr int kBfStages = 3, kBfLds = kBfStages * (64 + 128) * 128;

static __global__ __launch_bounds__(256, 2) void conv_block_fwd_kernel(const BlockFwdParams P) {
  extern __shared__ uint4 bf_lds[];
  __shared__ unsigned any_s[4], all_s[4];
  constexpr int NST = kBfStages, OPA = 64 * LDS_ROW_U4, OPB = 128 * LDS_ROW_U4;
  uint4* const lds = bf_lds;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  touch_args<(int)(sizeof(BlockFwdParams) / 64)>(P);
  // XCD x takes the x-th eighth of the tiles; the channels of a tile of positions follow each other and share its pixels in L2
  const int xcd = (int)blockIdx.x & 7, lo = (int)((long)xcd * P.total / 8), hi = (int)((long)(xcd + 1) * P.total / 8);
  const int L = lo + ((int)blockIdx.x >> 3);
  if (L >= hi) return;
  const int T = (int)fdiv((uint32_t)L, P.by_mt), row0 = (L - T * P.mt) * 64, j0 = T * 128;
  // the positions this lane fetches, and their kept channel groups (one bit each)
  constexpr int NB = DirectLoader<true, 128, 4>::NI;
  uint32_t voff[NB];
  unsigned kept[NB], any = 0, all = ~0u;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int q = imin(j0 + (wave * NB + j) * 8 + (lane >> 3), P.npix - 1);
    const int n = (int)fdiv((uint32_t)q, P.by_hw), p = q - n * P.HW, h = (int)fdiv((uint32_t)p, P.by_w), w = p - h * P.W_;
    voff[j] = (uint32_t)((n * P.HgWg + h * P.Wg + w) * P.Cp + DirectLoader<true, 128, 4>::chunk_k(lane, wave, j)) * 2u;
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
#pragma unroll
  for (int im = 0; im < 2; ++im)
#pragma unroll
    for (int in = 0; in < 4; ++in)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[im][in][v] = 0.0f;
  if (S > 0) {
    // step s = (kept channel group, tap); lane l keeps steps l and 64 + l
    auto entry = [&](int s) {
      const int i = s / taps, t = s - i * taps, r = t / P.kw;
      unsigned m = need;
      for (int k = i; k > 0; --k) m &= m - 1;
      return r | ((t - r * P.kw) << 4) | (__builtin_ctz(m | 0x80000000u) << 8);
    };
    const int e0 = entry(imin(lane, S - 1)), e1 = entry(imin(64 + lane, S - 1));
    DirectLoader<true, 64, 4> la;
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
    const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)lds);
    unsigned aaddr[2], baddr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 32 + (lane & 31), xr = (row & 7) ^ ((row >> 3) & 7);
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
    constexpr int LPS = 2 + NB;
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
  constexpr int PITCH = 136;  // (positions; rows 272 bytes apart)
#pragma unroll
  for (int im = 0; im < 2; ++im)
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const int row = im * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), col = wave * 32 + (lane & 31);
      tile[row * PITCH + col] = (uint16_t)words[im][v >> 1];
      tile[(row + 1) * PITCH + col] = (uint16_t)(words[im][v >> 1] >> 16);
    }
  // Where a group is kept for some positions only, the others multiplied its weights by zeros, which a weight that is not
  // finite makes NaN: such a result is summed again over the groups that its own position keeps.  (No finite sum had such a
  // term: two comparisons for every four results are all that is paid for it.)
  if (mixed && nan) {
    const int col = wave * 32 + (lane & 31), q = imin(j0 + col, P.npix - 1);
    const int n = (int)fdiv((uint32_t)q, P.by_hw), p = q - n * P.HW, h = (int)fdiv((uint32_t)p, P.by_w), w = p - h * P.W_;
    const uint8_t* const m = P.blk + ((long)n * P.RB + (int)fdiv((uint32_t)p, P.by_x)) * P.CB;
    const uint16_t* const at = P.grid + ((long)n * P.HgWg + h * P.Wg + w) * P.Cp;
#pragma unroll 1
    for (int i = 0; i < 32; ++i) {
      const int row = (i >> 4) * 32 + 8 * ((i >> 2) & 3) + 4 * (lane >> 5) + (i & 3);
      if ((tile[row * PITCH + col] & 0x7fff) <= 0x7f80 || row0 + row >= P.Cout) continue;
      const uint16_t* const wr = P.W + (long)(row0 + row) * P.ldw;
      float x = 0.0f;
#pragma unroll 1
      for (int cg = 0; cg < P.CG && x == x; ++cg) {
        if (!m[cg / P.cg_per_blk]) continue;
#pragma unroll 1
        for (int t = 0; t < taps; ++t) {
          const int r = t / P.kw, s = t - r * P.kw;
#pragma unroll 1
          for (int c = cg * 64; c < cg * 64 + 64; ++c)
            x += bf16_bits_to_f32(wr[t * P.Cp + c]) * bf16_bits_to_f32(at[(long)(r * P.Wg + s) * P.Cp + c]);
        }
      }
      tile[row * PITCH + col] = f32_to_bf16_bits(x);
    }
  }
  __syncthreads();
  // a thread takes E positions of a row: they lie in one plane (host: the planes are whole pieces)
  auto store = [&](auto unit) {
    using U = decltype(unit);
    constexpr int E = (int)sizeof(U) / 2, PR = 128 / E;  // positions per store, threads per row
    const int c = (tid % PR) * E, q = j0 + c;
    if (q >= P.npix) return;
    const int n = (int)fdiv((uint32_t)q, P.by_hw), p = q - n * P.HW;
    uint16_t* const out = P.Y + ((long)n * P.Cout + row0) * P.HW + p;
    for (int r = tid / PR; r < 64 && row0 + r < P.Cout; r += 256 / PR) *reinterpret_cast<U*>(out + (long)r * P.HW) = *reinterpret_cast<const U*>(tile + r * PITCH + c);
  };
  if (P.width == 16) store(uint4{});
  else if (P.width == 8) store(uint2{});
  else if (P.width == 4) store(uint32_t{});
  else store(uint16_t{});
}

// (conv_kept.hip)
int32_t launch_conv_block_fwd(const BlockFwdParams& P, hipStream_t stream);

}  // namespace ard
