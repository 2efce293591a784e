// LDS-direct bf16 path of the gathered GEMM for gfx950.
//
// Workgroup tiles BM x BN x 64 of 16x16x32 bf16 MFMA tiles: 256x256, 256x128, 128x256 with 8
// wavefronts (two per SIMD), 128x128, 128x64 and 64x64 with 4 wavefronts for products too small
// to fill 256 CUs with large tiles; optional split of the contraction over blockIdx.y with
// fp32 partial sums that a finishing kernel reduces (fixed split: deterministic).
//
// Operand staging uses LDS-direct loads (global_load_lds_dwordx4): a wavefront instruction
// moves 64 x 16 bytes from per-lane global addresses into 1 KiB of consecutive LDS with no
// register in between, so a whole stage stays in flight behind the MFMAs of the previous one.
// The LDS layout is therefore fixed by lane order, and each lane picks WHICH chunk it fetches
// so that the layout comes out swizzled (bank-conflict free for the fragment reads):
//   KC operand (contraction-contiguous in memory): LDS tile [rows][8 chunks of 16 B]; an
//     instruction fills 8 rows; lane = (row, slot) fetches logical chunk slot ^ xr(row).
//     Fragments: ds_read_b128.
//   MC operand (contraction-strided in memory): LDS tile [64 k][rows] exactly as in memory; lane
//     = (k, pos) fetches chunk pos ^ mc_swz(k).  Fragments: two ds_read_b64_tr_b16 (the
//     transposing LDS read of gfx950) per MFMA operand, no register transpose anywhere.
// LDS: [A stages | B stages] (2 stages, 3 for tiles of 64x64, 256x128 and 128x256); the stage is an immediate offset
// of the fragment reads, so every read address is a loop invariant.
//
// What bounds the large tiles is power and the way of the loads.  16x16x32 MFMAs take less power than 32x32x16 ones (random
// operands from registers, 300 launches in a row: 67 against 79 us for the FLOPs of a 4096^3 product, with the LDS reads of a
// 256 x 256 tile beside them 84 against 90).  Three stages of 48 KB give the loads two steps to arrive (a step of a 256 x 128
// tile is 1024 MFMA clocks, about what a load from the Infinity Cache takes), and issued as a burst the loads of a stage
// hold up the MFMAs behind them.  Medians of the kernels in whole training steps, with two stages of 32x32x16 MFMAs and so, traced in
// turn on one card, us: 4096^3, 64 x 64 tiles at dp = 2, forward 79 and 73, data gradient 93 and 80, weight gradient 88 and 83;
// 8192 x 2048 x 1024 to fp32 55 and 42, 8192 x 1024 x 2048 43 and 37; convolution products of 128 images of 28 x 28, 3 x 3: 128 -> 256
// channels 78 and 72 (256 x 256 tiles), its data gradient 72 and 62, weight gradient 73 and 66; listed pixels 60 and 51, 50 and 44.
//
// Tile patterns (Section 3.2) are period patterns over the linear tile index, so the tile
// rows (or columns) fall into a few CLASSES that share one kept-column (kept-row) set:
// class members, and the kept set of a class, are both arithmetic progressions.  A
// workgroup takes consecutive members of ONE class as its rows or columns and walks that
// class's kept set along the contraction, so dropped tiles cost nothing and the macro
// tile stays wide.  ClassTab carries the progressions.
//
// The same kernel runs the convolutions on a channels-last grid of the kept feature maps
// (MODE 1: rows of B are output pixels, contraction = (tap, channel); MODE 2: weight gradient,
// contraction over the grid's pixels).
//
// Restrictions checked on the host (anything else goes through gemm_kernel): bf16, 16-byte
// aligned operands, every extent along a 16-byte run a multiple of 8 (or zero-padded storage),
// contraction map = identity or a block progression with block size a multiple of 64.
#pragma once
#include <type_traits>
#include <utility>

#include "engine.hpp"

namespace ard {

constexpr int F_MAXCLS = 16;

struct ClassTab {
  int ncls;                       // 0: plain tiles_m x tiles_n grid over P.am / P.bn / P.k
  int nblk[F_MAXCLS];             // workgroups of class c
  int mblk[F_MAXCLS];             // workgroup rows of class c
  // row side (M): block progression off + i*step, `cnt` blocks of size bs (bs == 0: identity rows)
  int m_off[F_MAXCLS], m_cnt[F_MAXCLS], m_step, m_bs, m_phys;
  // column side (N)
  int n_off[F_MAXCLS], n_cnt[F_MAXCLS], n_step, n_bs, n_phys;
  // contraction side (K) (bs == 0: identity contraction P.k)
  int k_off[F_MAXCLS], k_cnt[F_MAXCLS], k_step, k_bs, k_phys;
};

// Implicit-GEMM convolution on a channels-last, zero-bordered copy of the activations
// T[(n*Hg + h)*Wg + w][Cp] (Cp channels per pixel, a multiple of 64): the patch of output pixel
// (n, ho, wo) and tap (r, s) is the Cp-run that starts at pixel (n*Hg + ho + r)*Wg + wo + s, so
// along the contraction k = (tap, c) every row of the im2col matrix is its base pixel plus an
// offset that depends on k only.
struct ConvMap {
  int HoWo, Wo;     // output pixels per image / per row
  int HgWg, Wg;     // pixels per image / per row of the bordered grid
  int Cp, kw;       // channels per pixel of the grid, taps per filter row
  int npix;         // output pixels over the batch (rows of the im2col matrix)
  int out_chan;     // channels per image of the output tensor (NCHW)
  const int* chan;  // optional: output channel of compact row i (kept-channel list), else i
  int n_rows;       // valid compact output rows (channels)
  // optional list of kept output pixels (row-based sensitivity-aware pattern, Section 5.2.1): compact
  // column j of the product is pixel pix[j] of the pix_total pixels; npix then counts the kept ones.
  // pix_fixed >= 0 (host-side bounds proof only): every column reads that pixel instead of the list.
  const int* pix;
  int pix_total, pix_fixed;
  int pix_pairs;  // list entries 2i, 2i+1 are pixels 2m, 2m+1 of one image (or both padding): the list holds runs, stored in pieces
  int taps;       // of the filter; it and what follows: set_divisors
  FastDiv per_img, per_row, by_cp, by_kw, by_taps;  // HoWo, Wo, Cp, kw, taps
  // Every lane finds its rows' pixels and every step its tap before anything is loaded: by division, a workgroup's first
  // load came 4000 of a 256 x 256 tile's 70000 clocks after its start.
  void set_divisors(int n_taps) {
    taps = n_taps;
    per_img = fast_div((uint32_t)HoWo), per_row = fast_div((uint32_t)Wo), by_cp = fast_div((uint32_t)Cp);
    by_kw = fast_div((uint32_t)kw), by_taps = fast_div((uint32_t)n_taps);
  }
};

// Weight gradient over listed output positions (MODE 3; row- and block-based sensitivity-aware patterns, Section 5.2):
// column block cb (a group of `chans` input channels over all taps, `cols` columns of the product, `tiles` column
// tiles) contracts over its own cnt[cb] output positions list[cb * stride ...], numbered n * HoWo + p.
struct ListMap {
  int ncls;          // 0 (shares its place with ClassTab::ncls)
  int stride, max;   // entries reserved per block; a count beyond `max` is cut
  int tiles, cols, chans, cols_per_tap;
  int pad;           // grid pixel whose gradient is zero: fills up the last step
  const int* list;
  const int* cnt;
};

// Dropped tiles of a tile-masked output (MODE 0, weight gradient): zeroed by the last `blocks` workgroups of the launch
struct ZeroTilesJob {
  int blocks, rows, cols, TC, dp, o;
  FastDiv by_tr, by_tc, by_chunks;  // tile rows, tile columns / 8, cols / 8
};

// (What every launch reads comes first and is fetched in one go, see touch_args; the class tables come last.)
struct FastParams {
  const uint16_t* A;
  const uint16_t* B;
  uint16_t* C;
  int lda, ldb, ldc;
  int ncls;               // tab.ncls (set_bands)
  int M, N, tiles_m, tiles_n, group_m, total_tiles;
  int splits;
  FastDiv tiles_div, band_div;  // total_tiles, group_m * tiles_n (set_bands)
  float alpha, beta;
  Axis am, bn, k;  // plain mode: compact -> physical rows of A (M), rows of B (N), contraction
  float* part;               // != NULL: write fp32 partial sums part[split][M][N] instead of C
  const uint16_t* relu_src;  // optional, same layout as C
  int relu, out_f32;
  int c_rows_mapped, c_cols_mapped;  // output rows / columns go through the M / N map (else identity); M x N of them exist
  // Scattering epilogue (row patterns without compact outputs): the tile's results go through
  // LDS and are written, with the dropped positions it owns as +0.0, through these affine maps.
  int scatter;
  int scatter_rows_only;  // the tile writes its kept rows only (a separate pass zeroes the dropped rows)
  Axis srm, scn;
  // MODE 1, optional (block-based sensitivity-aware pattern, Section 5.2.2): the column tile t of the
  // product contracts over the kb_cnt[t] 64-wide blocks kb_list[t * kb_stride ...] of the contraction only
  // (at most 128 of them); entries of cv.pix may then be -1 (padding of a tile: nothing is stored).
  const int* kb_list;
  const int* kb_cnt;
  int kb_stride;
  union {
    ConvMap cv;  // MODE 1 / 2 / 3 of the kernel only
    ZeroTilesJob zt;
  };
  long a_elems, b_elems;  // elements the caller owns behind A / B: what the loaders may touch (host-side proof)
  union {
    ClassTab tab;
    ListMap li;  // MODE 3
  };
};

// Brings the first LINES 64-byte lines of a kernel's arguments into the scalar cache with one round trip.  Left
// to themselves the loads come in small groups behind branches, each a trip of about 1000 clocks to memory the
// host has just written: 5 of the 17 thousand clocks of a 1024 x 1024 x 1024 product on 64 x 64 tiles.
template <int LINES, class Params>
__device__ __forceinline__ void touch_args(const Params& P) {
  const int* w = reinterpret_cast<const int*>(&P);
  int x = 0;
#pragma unroll
  for (int i = 0; i < LINES; ++i) x |= w[16 * i];
  asm volatile("" ::"s"(x));
}

// Two fp32 values to packed bf16 (low half = first) with the conversion instruction of gfx950
// (round to nearest even, the same rounding as f32_to_bf16_bits for finite values).
typedef __bf16 bf16x2_hw_t __attribute__((ext_vector_type(2)));
typedef float f32x2_hw_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_hw_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_hw_t));
}

#define ARD_LDS_PTR(p) ((void __attribute__((address_space(3)))*)(p))
#define ARD_GLB_PTR(p) ((const void __attribute__((address_space(1)))*)(p))

// four words at any word address
struct U4AnyWord {
  uint32_t x, y, z, w;
};

// 64 zero bytes: source of the chunks that lie beyond the end of the contraction
static __device__ uint4 g_zero_chunk[4];

// physical start of the 64-wide contraction slab that begins at compact index ks (uniform)
__host__ __device__ __forceinline__ int fast_kslab(const Axis& k, int ks) {
  if (k.kind == AX_AFFINE) return k.off + ks;
  const int q = ks / k.bs;
  if (k.kind == AX_BAFF) return (k.off + q * k.step) * k.bs + (ks - q * k.bs);
  return (k.list[q] + k.off) * k.bs + (ks - q * k.bs);
}

// A contraction axis made of 32-wide blocks in arithmetic progression (the paper's 32 x 32 tiles): a
// 64-deep step holds two kept blocks, `step` blocks apart in memory.  The slab of a step starts at its
// first block; the lanes that fetch the step's upper half add this constant (in contraction elements) to
// their offset once, at set-up, so the loop itself does not change.
__host__ __device__ __forceinline__ int direct_kbump(const Axis& k) {
  return (k.kind == AX_BAFF && k.bs == 32) ? (k.step - 1) * 32 : 0;
}

// KC tile: chunk c of row r sits at position c ^ kc_swz(r).  A 16-byte LDS read serves 16 lanes at a time, lanes 0-3, 12-15,
// 20-23 and 24-27 first: for MFMA tiles of 16 rows (lane l: row l % 16, chunk l / 16) these are eight rows of one chunk and eight
// of its neighbour, for tiles of 32 rows (T32) sixteen rows of one chunk.
template <bool T32>
__host__ __device__ __forceinline__ int kc_swz(int row) {
  return T32 ? (row & 7) ^ ((row >> 3) & 7) : row & 6;
}

template <bool KC, int ROWS, int NW, bool T32 = false> struct DirectLoader;

// Both loaders keep, per lane and instruction, a loop-invariant 32-bit BYTE offset from a base that
// is uniform over the workgroup; a contraction step only moves the uniform base, so a load costs
// no vector ALU work.  A lane whose tile row lies beyond the operand reads some valid row instead
// (clamped at set-up): such rows only feed outputs that are never stored, or that the epilogue
// overwrites with zeros.  Only the last, partial step of a contraction redirects lanes to a zero chunk.
template <int ROWS, int NW, bool T32> struct DirectLoader<true, ROWS, NW, T32> {
  static constexpr int NI = ROWS / 8 / NW;  // instructions per wavefront and stage (8 rows each)
  static_assert(NI >= 1, "tile too small for the workgroup");
  const char* base;
  uint32_t voff[NI];
  __host__ __device__ static __forceinline__ int chunk_k(int lane, int wave, int j) {
    const int row = (wave * NI + j) * 8 + (lane >> 3);
    return ((lane & 7) ^ kc_swz<T32>(row)) * 8;
  }
  // (host-callable: the host-side bounds proof runs this very arithmetic for every lane)
  __host__ __device__ __forceinline__ void init(const uint16_t* p, int ld, const Axis& r, int row0, int lane, int wave,
                                                int kbump = 0) {
    base = reinterpret_cast<const char*>(p);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int row = imin(row0 + (wave * NI + j) * 8 + (lane >> 3), r.n - 1);
      // (a block axis counts its last block in full even when the operand ends inside it)
      int prow = ax_phys(r, row);
      if (r.kind == AX_BLOCK || r.kind == AX_BAFF) prow = imin(prow, r.nphys - 1);
      const int ck = chunk_k(lane, wave, j);
      voff[j] = (uint32_t)(prow * ld + ck + (ck >= 32 ? kbump : 0)) * 2u;
    }
  }
  // rows = output pixels of a convolution: base pixel of the patch in the bordered grid
  __host__ __device__ __forceinline__ void init_pixels(const uint16_t* p, const ConvMap& cv, int row0, int lane, int wave) {
    base = reinterpret_cast<const char*>(p);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      int row = imin(row0 + (wave * NI + j) * 8 + (lane >> 3), cv.npix - 1);
      if (cv.pix_fixed >= 0) row = cv.pix_fixed;
      else if (cv.pix) row = imax(cv.pix[row], 0);  // (-1: padding entry, reads pixel 0, stores nothing)
      const int n = (int)fdiv((uint32_t)row, cv.per_img), rem = row - n * cv.HoWo;
      const int ho = (int)fdiv((uint32_t)rem, cv.per_row), wo = rem - ho * cv.Wo;
      voff[j] = (uint32_t)((n * cv.HgWg + ho * cv.Wg + wo) * cv.Cp + chunk_k(lane, wave, j)) * 2u;
    }
  }
  // full step: nothing but the loads
  __device__ __forceinline__ void issue(uint4* op_tile, int kslab, int wave) const {
    const char* sb = base + (long)kslab * 2;  // uniform
#pragma unroll
    for (int j = 0; j < NI; ++j)
      __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(sb + voff[j]), ARD_LDS_PTR(op_tile + (wave * NI + j) * 64), 16, 0, 0);
  }
  // one of the NI loads of a full step (for callers that spread them between other instructions)
  __device__ __forceinline__ void issue_one(uint4* op_tile, int kslab, int wave, int j) {
    const char* sb = base + (long)kslab * 2;
    asm volatile("" : "+v"(voff[j]));  // (widened ahead of the loop, it would be added to the base by the vector unit instead of the load)
    __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(sb + voff[j]), ARD_LDS_PTR(op_tile + (wave * NI + j) * 64), 16, 0, 0);
  }
  // last, partial step of a contraction: chunks beyond its end come from the zero chunk
  __host__ __device__ static __forceinline__ bool tail_live(int lane, int wave, int j, int kslab, int krem, int kphys_end,
                                                            int kbump = 0) {
    const int k = chunk_k(lane, wave, j);
    return k < krem && kslab + k + (k >= 32 ? kbump : 0) + 8 <= kphys_end;
  }
  // byte offset from the operand's base of instruction j's chunk in the step whose slab starts at kslab
  __host__ __device__ __forceinline__ long byte_offset(int j, int kslab) const { return (long)kslab * 2 + voff[j]; }
  __device__ __forceinline__ void issue_tail(uint4* op_tile, int kslab, int krem, int kphys_end, int lane, int wave,
                                             int kbump = 0) const {
    asm volatile("; partial contraction step" ::: "memory");  // keeps this path out of the full step's code
    const char* sb = base + (long)kslab * 2;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const char* src = sb + voff[j];
      if (!tail_live(lane, wave, j, kslab, krem, kphys_end, kbump)) src = reinterpret_cast<const char*>(g_zero_chunk);
      __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(src), ARD_LDS_PTR(op_tile + (wave * NI + j) * 64), 16, 0, 0);
    }
  }
};

// swizzle of an MC tile: chunk c of contraction row k sits at position c ^ mc_swz(k).  Rows are
// ROWS*2 bytes apart; the XOR makes the eight rows that 32 lanes of a transposing read touch (k .. k + 3 and k + 8 .. k + 11,
// 32 bytes of each) land in different banks (rows of 256+ bytes all start at the same bank, rows of 128 bytes alternate).
template <int ROWS>
__host__ __device__ __forceinline__ int mc_swz(int k) {
  return (ROWS >= 128 ? 4 * (k & 3) : 4 * ((k >> 1) & 1)) + 2 * ((k >> 3) & 1);
}

template <int ROWS, int NW, bool T32> struct DirectLoader<false, ROWS, NW, T32> {
  static constexpr int CPR = ROWS / 8;         // 16-byte chunks per contraction row
  static constexpr int KPI = 64 / CPR;         // contraction rows per instruction
  static constexpr int NI = 64 / KPI / NW;     // instructions per wavefront and stage
  static_assert(NI >= 1, "tile too small for the workgroup");
  const char* base;
  int ld;
  uint32_t voff[NI];  // (contraction row within the step) * ld + column of this lane's chunk, in bytes
  __host__ __device__ __forceinline__ int lane_chunk(int lane, int wave, int j) const {
    const int kloc = KPI * (wave * NI + j) + lane / CPR;
    return (lane % CPR) ^ mc_swz<ROWS>(kloc);
  }
  __host__ __device__ __forceinline__ void init(const uint16_t* p, int ld_, const Axis& r, int row0, int lane, int wave,
                                                int kbump = 0) {
    base = reinterpret_cast<const char*>(p);
    ld = ld_;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int kl = KPI * (wave * NI + j) + lane / CPR;
      const int kloc = kl + (kl >= 32 ? kbump : 0);
      const int col = imin(row0 + lane_chunk(lane, wave, j) * 8, r.n - 8);  // runs beyond the axis: clamped
      // (a block axis counts its last block in full even when the operand ends inside it)
      int pcol = ax_phys(r, col);
      if (r.kind == AX_BLOCK || r.kind == AX_BAFF) pcol = imax(imin(pcol, (r.nphys - 8) & ~7), 0);
      voff[j] = (uint32_t)(kloc * ld + pcol) * 2u;
    }
  }
  // columns = (tap, channel) of the weight gradient: pixel offset of the tap plus the channel
  __host__ __device__ __forceinline__ void init_tap_columns(const uint16_t* p, const ConvMap& cv, int ncols, int row0,
                                                            int lane, int wave) {
    base = reinterpret_cast<const char*>(p);
    ld = cv.Cp;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int kloc = KPI * (wave * NI + j) + lane / CPR;
      const int col = imin(row0 + lane_chunk(lane, wave, j) * 8, ncols - 8);
      const int t = (int)fdiv((uint32_t)col, cv.by_cp), r = (int)fdiv((uint32_t)t, cv.by_kw);
      voff[j] = (uint32_t)(kloc * ld + (r * cv.Wg + t - r * cv.kw) * cv.Cp + (col - t * cv.Cp)) * 2u;
    }
  }
  __device__ __forceinline__ void issue(uint4* op_tile, int kslab, int wave) const {
    const char* sb = base + (long)kslab * ld * 2;  // uniform
#pragma unroll
    for (int j = 0; j < NI; ++j)
      __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(sb + voff[j]), ARD_LDS_PTR(op_tile + (wave * NI + j) * 64), 16, 0, 0);
  }
  __device__ __forceinline__ void issue_one(uint4* op_tile, int kslab, int wave, int j) {
    const char* sb = base + (long)kslab * ld * 2;
    asm volatile("" : "+v"(voff[j]));
    __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(sb + voff[j]), ARD_LDS_PTR(op_tile + (wave * NI + j) * 64), 16, 0, 0);
  }
  __host__ __device__ static __forceinline__ bool tail_live(int lane, int wave, int j, int kslab, int krem, int kphys_end,
                                                            int kbump = 0) {
    const int kloc = KPI * (wave * NI + j) + lane / CPR;
    return kloc < krem && kslab + kloc + (kloc >= 32 ? kbump : 0) < kphys_end;
  }
  __host__ __device__ __forceinline__ long byte_offset(int j, int kslab) const { return (long)kslab * ld * 2 + voff[j]; }
  __device__ __forceinline__ void issue_tail(uint4* op_tile, int kslab, int krem, int kphys_end, int lane, int wave,
                                             int kbump = 0) const {
    asm volatile("; partial contraction step" ::: "memory");
    const char* sb = base + (long)kslab * ld * 2;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const char* src = sb + voff[j];
      if (!tail_live(lane, wave, j, kslab, krem, kphys_end, kbump)) src = reinterpret_cast<const char*>(g_zero_chunk);
      __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(src), ARD_LDS_PTR(op_tile + (wave * NI + j) * 64), 16, 0, 0);
    }
  }
};

// MC operand whose contraction rows are listed grid pixels (MODE 3): the list of the steps in flight lies in LDS as
// pixel numbers, a lane looks up the rows of its chunks one step before it loads them.
template <int ROWS, int NW> struct ListLoader {
  using L = DirectLoader<false, ROWS, NW>;
  static constexpr int NI = L::NI;
  const char* base;
  uint32_t row_bytes;
  uint32_t coff[NI];  // this lane's chunk within a pixel (a tap's pixel offset included), in bytes
  int kloc[NI];       // contraction row within the step
  __host__ __device__ __forceinline__ void init(const uint16_t* p, int ld, int ncols, int col0, int lane, int wave) {
    base = reinterpret_cast<const char*>(p);
    row_bytes = (uint32_t)ld * 2u;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      kloc[j] = L::KPI * (wave * NI + j) + lane / L::CPR;
      coff[j] = (uint32_t)imin(col0 + ((lane % L::CPR) ^ mc_swz<ROWS>(kloc[j])) * 8, ncols - 8) * 2u;
    }
  }
  // columns = (tap, channel of the block)
  __host__ __device__ __forceinline__ void init_taps(const uint16_t* p, const ConvMap& cv, const ListMap& li, int cb, int col0, int lane, int wave) {
    init(p, cv.Cp, li.cols, col0, lane, wave);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int col = (int)(coff[j] >> 1), t = col / li.cols_per_tap, r = (int)fdiv((uint32_t)t, cv.by_kw);
      coff[j] = (uint32_t)((r * cv.Wg + t - r * cv.kw) * cv.Cp + cb * li.chans + col - t * li.cols_per_tap) * 2u;
    }
  }
  __device__ __forceinline__ void look(const int* step_list, uint32_t (&off)[NI]) const {
#pragma unroll
    for (int j = 0; j < NI; ++j) off[j] = __umul24((uint32_t)step_list[kloc[j]], row_bytes) + coff[j];
  }
  __device__ __forceinline__ void issue_one(uint4* op_tile, uint32_t off, int wave, int j) const {
    __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(base + off), ARD_LDS_PTR(op_tile + (wave * NI + j) * 64), 16, 0, 0);
  }
};
// list entries a workgroup of the 256-row / 128-row tile holds in LDS at a time
constexpr int direct_list_cap(int bm) { return bm == 256 ? 4096 : 3072; }

// Byte offset, inside an MC operand tile of `ROWS` rows, of this lane's source position for the
// transposing reads of the 16-wide MFMA tile that starts at tile row `tile_col0`.  The reads
// of slice q, half h add the immediate (q*32 + h*4) * ROWS*2.
// ds_read_b64_tr_b16 works on groups of 16 lanes: result lane i, element e comes from source
// lane 4e + i/4, element i%4.  With source lane s at (k = s/4, column 4*(s%4)) of a 4 x 16
// block, result lane i holds column i for k = 0..3: the MFMA operand order.
template <int ROWS>
__device__ __forceinline__ int mc_frag_base(int tile_col0, int lane) {
  const int s = lane & 15, k = (lane >> 4) * 8 + (s >> 2);
  const int pc = ((tile_col0 >> 3) + ((s & 3) >> 1)) ^ mc_swz<ROWS>(k);
  return k * (ROWS * 2) + pc * 16 + 8 * (s & 1);
}

// LDS fragment reads are issued as volatile asm with ONE explicit wait per unit (a 32-wide slice of a step by a part of the
// wavefront's rows or columns): the compiler cannot sink a read next to its consumer, so a unit's reads are in flight while
// the MFMAs of the one before run (left to itself the scheduler waits right after each read).
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
struct Frag {  // one MFMA operand: a full 16-byte read (KC) or two transposing 8-byte reads (MC)
  u32x4_t v;
  u32x2_t lo, hi;
};
template <int OFF>
__device__ __forceinline__ void lds_read_b128(u32x4_t& dst, unsigned byte_addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(byte_addr), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void lds_read_tr16_b64(u32x2_t& dst, unsigned byte_addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(byte_addr), "n"(OFF));
}
template <bool KC>
__device__ __forceinline__ void frag_wait(Frag& f) {
  // tie the destination registers to the wait so no consumer can be scheduled before it
  if (KC) asm volatile("" : "+v"(f.v));
  else asm volatile("" : "+v"(f.lo), "+v"(f.hi));
}
template <bool KC>
__device__ __forceinline__ bf16x8_t frag_value(const Frag& f) {
  if (KC) return __builtin_bit_cast(bf16x8_t, f.v);
  u32x4_t t = {f.lo[0], f.lo[1], f.hi[0], f.hi[1]};
  return __builtin_bit_cast(bf16x8_t, t);
}

// LDS stages of a tile configuration: the loads of NST - 1 contraction steps are in flight
// while one step is multiplied.  A 4-wavefront workgroup wants a second workgroup on its CU
// (8 wavefronts hide the LDS and MFMA latencies), so its stages must fit twice into the 160 KiB
// LDS; only the smallest of these tiles has room for a third stage.  Of the 8-wavefront tiles, one workgroup a CU, those of 384
// rows and columns together have it (two stages: 8192 x 2048 x 1024 42 us, three 37).
constexpr int direct_stages(int bm, int bn) { return bm + bn <= 128 || bm + bn == 384 ? 3 : 2; }
// MFMAs of a wavefront, from the hand-over of a stage on, over which the loads of a stage are spread (`step`: of a step, `unit`: of a
// unit; the last unit of a step but one is left out).  Over all of a step where a stage has two steps to arrive; where it has one,
// what a spread gains at the issue it loses at the end: over five eighths of a step, 4096^3 at dp = 2 took 134 instead of 120
// thousand clocks on 256 x 256 tiles, and a unit is best for 128 x 128.  128 x 448, whose units are four MFMAs: half a step 62 us, one
// unit 66 (above).  Small tiles: a whole step made five dependent launches of 64 x 64 tiles 56.3 us instead of 55.
constexpr int direct_load_window(int bm, int bn, int step, int unit) {
  return bm + bn == 384 ? step - unit : bn == 448 ? step / 2 : bm + bn >= 512 ? 2 * unit : unit;
}
// Wavefronts side by side along the columns, so that each has whole 32 x 32 tiles
constexpr int direct_wave_columns(int bn, int nw) { return nw == 8 && (bn == 256 || bn == 384) ? 4 : 2; }
// Bytes between the rows of a tile on its way out through LDS, in elements of `size` bytes: the rows that a store to LDS
// touches at a time start four banks apart.
constexpr int direct_pitch(int bn, int size) { return bn * size + 16; }
// Dynamic LDS of a product: the operand stages (MODE 3: and the steps' pixels), or the output tile (as bf16, or
// half of it as fp32, which is no more) and its rows' places if that is more.
constexpr size_t direct_lds_bytes(int bm, int bn, int mode) {
  const size_t stages = (size_t)direct_stages(bm, bn) * (bm + bn) * LDS_ROW_U4 * sizeof(uint4) + (mode == 3 ? direct_list_cap(bm) * 4 : 0);
  const size_t tile = (size_t)bm * direct_pitch(bn, 2) + (size_t)bm * 4;
  return tile > stages ? tile : stages;
}

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(const F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(const F& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Stages of `bytes` bytes whose fragments, up to `reach` bytes behind a place in the first, are within the 16 bits of an LDS
// read's offset
constexpr int frag_stages(int bytes, int reach) { return reach + 2 * bytes <= 65535 ? 3 : reach + bytes <= 65535 ? 2 : 1; }

// Plain barrier.  The LDS stages are filled by LDS-direct loads (each wave waits for its own
// with wait_vmcnt before the barrier) and read by volatile asm, so no fence is wanted: a fence
// would also wait for the younger stages still in flight.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Scattering store of one workgroup tile.  Output maps are affine with off < step: compact index i owns the
// physical group [i*step, (i+1)*step) that contains its kept position, the last index also the tail up to nphys;
// everything in the owned region that is not a kept position is written as +0.0.
// `img` holds the image of compact rows [m0, m1) in LDS exactly as it leaves: physical columns with their zeros,
// `pitch` elements per row, shifted so that the 16-byte pieces of a row in LDS are the 16-byte pieces of its
// place in memory (rows may have any length and alignment).  A row leaves piece by piece, only those its region
// cuts at either end element by element.
__device__ __forceinline__ int scatter_shift(const FastParams& P, int r, int c_lo) {
  return (int)(((reinterpret_cast<uintptr_t>(P.C) >> 1) + (uintptr_t)((long)r * P.ldc + c_lo)) & 7);
}
__device__ __forceinline__ void direct_scatter_rows(const uint4* img, int pitch, const FastParams& P, int m0, int m1, int c_lo,
                                                    int c_hi, int tid, int nthreads) {
  const Axis& rm = P.srm;
  const int CW = (c_hi - c_lo + 14) >> 3;  // (most pieces a row can have)
  // rows to write: the kept ones alone, or with the dropped ones of their groups, and after the last group the rest
  const bool all = !P.scatter_rows_only;
  const int sr = all ? rm.step : 1;
  const int r_first = all ? m0 * sr : m0 * rm.step + rm.off, r_inc = all ? 1 : rm.step;
  const int nrows = all ? (m1 == P.M ? rm.nphys : m1 * sr) - r_first : m1 - m0;
  const int total = nrows * CW;
  const float inv_cw = 1.0f / (float)CW, inv_sr = 1.0f / (float)sr;  // (indices below 2^20: (i + 1/2) / n truncates exactly)
  constexpr int U = 4;  // pieces in flight per thread
  for (int e0 = tid; e0 < total; e0 += U * nthreads) {
    uint4 v[U];
    long at[U];   // element index of the piece in C
    int c0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = imin(e0 + u * nthreads, total - 1);
      const int q = (int)(((float)e + 0.5f) * inv_cw), cq = e - q * CW;
      const int i = (int)(((float)q + 0.5f) * inv_sr), g = q - i * sr;
      const int r = r_first + q * r_inc;
      uint32_t m = (!all || g == rm.off) && i < m1 - m0 ? ~0u : 0u;
      asm("" : "+v"(m));  // (kept as a mask: behind a branch every LDS read would be waited for by itself)
      v[u] = img[imin(i, m1 - m0 - 1) * (pitch >> 3) + cq];
      v[u].x &= m, v[u].y &= m, v[u].z &= m, v[u].w &= m;
      c0[u] = c_lo - scatter_shift(P, r, c_lo) + cq * 8;
      at[u] = (long)r * P.ldc + c0[u];
      if (e0 + u * nthreads >= total) c0[u] = c_hi;  // nothing to store
    }
    if (P.relu_src) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (c0[u] >= c_hi) continue;
        const uint16_t* g = P.relu_src + at[u];
        uint16_t q[8];
        if (c0[u] >= c_lo && c0[u] + 8 <= c_hi && (reinterpret_cast<uintptr_t>(g) & 15) == 0) {
          *reinterpret_cast<uint4*>(q) = *reinterpret_cast<const uint4*>(g);
        } else {
#pragma unroll
          for (int t = 0; t < 8; ++t) q[t] = g[imin(imax(t, c_lo - c0[u]), c_hi - 1 - c0[u])];
        }
        uint32_t* w = reinterpret_cast<uint32_t*>(&v[u]);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          w[t] &= (bf16_bits_to_f32(q[2 * t]) > 0.0f ? 0xffffu : 0u) | (bf16_bits_to_f32(q[2 * t + 1]) > 0.0f ? 0xffff0000u : 0u);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c0[u] >= c_hi) continue;
      uint16_t* o = P.C + at[u];
      if (c0[u] >= c_lo && c0[u] + 8 <= c_hi) {
        *reinterpret_cast<uint4*>(o) = v[u];
      } else {
        const uint32_t* w = reinterpret_cast<const uint32_t*>(&v[u]);
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (c0[u] + t >= c_lo && c0[u] + t < c_hi) o[t] = (uint16_t)(w[t >> 1] >> (16 * (t & 1)));
      }
    }
  }
}
// Widest column step the LDS image is made for; wider ones go through partial sums and a finishing pass.  The image of a
// 128 x 128 tile holds 16 rows up to step 15, but beyond 8 it no longer pays: over 90 products with periods 9 .. 15
// (512 - 4096 rows, 1024 - 4096 units, bf16) image / pass is 1.005 in the geometric mean, the image ahead in 26 and behind
// in 29 by more than 3 % (4096^3, dp 2 x 12, weight gradient: 46 against 54 us; 4096 x 2048 x 2048, dp 1 x 15: 34 against 25).
constexpr int kScatterMaxStep = 8;

// What one workgroup computes: its row / column / contraction maps (class-based launches build them
// from the class tables), the first compact row and column of its tile and its share of the
// contraction.  Shared by the kernel and by the host-side bounds proof.
struct DirectWork {
  Axis am, bn, kax;
  int m0, n0, split;
};
// The `i`-th run of W rows (columns) of a class: whole blocks of the progression, or, where a block is wider
// than the tile, the i-th part of a block.  false: the run lies beyond the matrix.
template <int W>
__host__ __device__ __forceinline__ bool class_rows(int off, int cnt, int step, int bs, int phys, int i, Axis& r) {
  if (bs <= W) {
    const int g = W / bs, left = cnt - i * g;
    r = axis_baff(off + i * g * step, step, bs, left < g ? left : g, phys);
    return true;
  }
  const int parts = bs / W, m = i / parts, first = (off + m * step) * bs + (i - m * parts) * W;
  r = Axis{nullptr, AX_AFFINE, first, 1, 1, imin(W, phys - first), phys};
  return r.n > 0;
}
template <int F_BM, int BN, class Params>
__host__ __device__ __forceinline__ bool direct_assign(const Params& P, int block_id, DirectWork& w) {
  // Workgroup ids go round-robin over the 8 XCDs.  XCD x = id % 8 takes, of every class, the
  // contiguous share [x*n/8, (x+1)*n/8) of its n workgroups: the shares are compact rectangles
  // (operand panels stay in that XCD's L2) and heavy and light classes are spread evenly.
  const int xcd = block_id & 7;
  int local = block_id >> 3;
  Axis am = P.am, bn = P.bn, kax = P.k;
  int m0 = 0, n0 = 0;
  int split = 0;  // share of the contraction this workgroup takes
  if (P.ncls == 0) {
    // work items = (split, tile), split-major: an XCD's contiguous share holds whole splits (or long
    // runs of one), so the workgroups in flight on it read the same slab of the contraction
    const int total = P.total_tiles * P.splits;
    const int lo = (int)((long)xcd * total / 8), hi = (int)((long)(xcd + 1) * total / 8);
    if (local >= hi - lo) return false;
    int L = lo + local;
    split = (int)fdiv((uint32_t)L, P.tiles_div);
    L -= split * P.total_tiles;
    // bands of group_m (a power of two) tile rows, walked column by column
    const int band = (int)fdiv((uint32_t)L, P.band_div), inb = L - band * P.group_m * P.tiles_n;
    const int rows_in_band = imin(P.group_m, P.tiles_m - band * P.group_m);
    int col;
    if (rows_in_band == P.group_m) col = inb >> (31 - __builtin_clz((unsigned)P.group_m));
    else col = inb / rows_in_band;
    m0 = (band * P.group_m + inb - col * rows_in_band) * F_BM;
    n0 = col * BN;
    // per-tile contraction lists: the length comes from the tile's count, the blocks are looked up step
    // by step (the host-side proof clears kb_cnt and walks the whole contraction, which bounds every list)
    if (P.kb_cnt) kax.n = imin(imax(P.kb_cnt[n0 / BN], 0), imin(kax.nphys / 64, 128)) * 64;
  } else {
    const ClassTab& t = P.tab;
    int c = 0, l = -1;
    for (; c < t.ncls; ++c) {
      const int lo = (int)((long)xcd * t.nblk[c] / 8), hi = (int)((long)(xcd + 1) * t.nblk[c] / 8);
      if (local < hi - lo) {
        l = lo + local;
        break;
      }
      local -= hi - lo;
    }
    if (l < 0) return false;
    // bands of group_m row blocks, walked column by column (as in the plain case): an XCD's share
    // of a class is about square, so its operand panels are reused out of that XCD's L2
    const int nbc = t.nblk[c] / t.mblk[c];
    const int band_sz = P.group_m * nbc;
    const int band = l / band_sz, inb = l - band * band_sz;
    const int rows_in_band = imin(P.group_m, t.mblk[c] - band * P.group_m);
    const int mi = band * P.group_m + inb % rows_in_band, ni = inb / rows_in_band;
    if (t.m_bs) {
      if (!class_rows<F_BM>(t.m_off[c], t.m_cnt[c], t.m_step, t.m_bs, t.m_phys, mi, am)) return false;
    } else {
      m0 = mi * F_BM;
    }
    if (!class_rows<BN>(t.n_off[c], t.n_cnt[c], t.n_step, t.n_bs, t.n_phys, ni, bn)) return false;
    if (t.k_bs) kax = axis_baff(t.k_off[c], t.k_step, t.k_bs, t.k_cnt[c], t.k_phys);
  }
  w.am = am, w.bn = bn, w.kax = kax;
  w.m0 = m0, w.n0 = n0, w.split = split;
  return true;
}

// Physical start of the contraction slab of absolute step s: `ks` along the A operand, `ksb` along B
// (MODE 1: slab (tap, c0) of the im2col row = offset of the tap's pixel plus the channel).
template <int MODE>
__host__ __device__ __forceinline__ void direct_slab(const FastParams& P, const Axis& kax, int s, int& ks, int& ksb) {
  if constexpr (MODE == 1) {
    // The steps run channel group by channel group, all taps of a group in a row: consecutive steps then read
    // the same 128 bytes of pixels that lie a few positions apart, nearly all of them lines the step before
    // left in L2 (tap by tap, a whole pass over the tile's channels lies between two reads of a line).
    const int cg = (int)fdiv((uint32_t)s, P.cv.by_taps), t = s - cg * P.cv.taps, r = (int)fdiv((uint32_t)t, P.cv.by_kw);
    ks = t * P.cv.Cp + cg * 64;
    ksb = (r * P.cv.Wg + t - r * P.cv.kw) * P.cv.Cp + cg * 64;
    return;
  }
  ks = fast_kslab(kax, s * 64);
  ksb = ks;
}

// May only the last step of this contraction be a partial one?  (The axis is affine, or made of whole blocks that hold whole steps.)
__host__ __device__ __forceinline__ bool direct_full_steps(const Axis& k) {
  return k.kind == AX_AFFINE || (k.kind == AX_BAFF && (k.bs % 64 == 0 || k.bs == 32) && k.nphys % k.bs == 0);
}

// The slabs of direct_slab one after the other from step `s` on, without the divisions that finding one takes; in scalar
// registers, so that the loads take their base from there.  (Host-callable: the bounds proof steps it beside direct_slab.)
template <int MODE> struct DirectSlabs {
  int at = 0, atb = 0, in_run = 0, run = 0, jump = 0, in_row = 0;
  __host__ __device__ static __forceinline__ int uniform(int x) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_readfirstlane(x);
#else
    return x;
#endif
  }
  __host__ __device__ __forceinline__ void begin(const FastParams& P, const Axis& kax, int s) {
    if constexpr (MODE == 1) {
      int ks, ksb;
      direct_slab<MODE>(P, kax, s, ks, ksb);
      at = uniform(ks), atb = uniform(ksb);
      in_run = s - (int)fdiv((uint32_t)s, P.cv.by_taps) * P.cv.taps, in_row = in_run - (int)fdiv((uint32_t)in_run, P.cv.by_kw) * P.cv.kw;
    } else {
      at = uniform(fast_kslab(kax, s * 64));
      run = kax.kind == AX_BAFF ? imax(kax.bs, 64) : 0x40000000, jump = kax.kind == AX_BAFF ? (kax.step - 1) * run : 0;
      in_run = kax.kind == AX_BAFF ? s * 64 % run : 0;
    }
  }
  __host__ __device__ __forceinline__ void next(const FastParams& P, int& ks, int& ksb) {
    if constexpr (MODE == 1) {
      ks = at, ksb = atb;
      at += P.cv.Cp, atb += P.cv.Cp;
      if (++in_row == P.cv.kw) in_row = 0, atb += (P.cv.Wg - P.cv.kw) * P.cv.Cp;
      if (++in_run == P.cv.taps) {  // the next 64 channels
        at += 64 - P.cv.taps * P.cv.Cp;
        atb = at;
        in_run = 0;
      }
    } else {
      ks = ksb = at;
      at += 64, in_run += 64;
      if (in_run == run) at += jump, in_run = 0;
    }
  }
};

// MODE 0: plain product.  MODE 1: convolution, B rows are output pixels gathered from the
// bordered channels-last grid (contraction = (tap, channel)), output NCHW.  MODE 2: weight
// gradient of the convolution, contraction over the grid's pixels, B columns = (tap, channel).
// MODE 3: the same over listed pixels (ListMap): what a pattern drops is neither loaded nor multiplied.  N=128,
// C=Cout=256, 28x28, 3x3, 30 % of the positions kept: 123 -> 42 us (row pattern), 4 x 38 -> 45 us (block pattern, four
// groups of channels).
// (body of the kernel as a device function: the grouped kernel of gemm.hip runs it on a range of
// its workgroups; block_id is the workgroup's index within the product, lds its dynamic LDS)
template <bool A_KC, bool B_KC, int F_BM, int BN, int NW, int MODE = 0>
__device__ __forceinline__ void direct_body(const FastParams& P, const int block_id, uint4* const lds) {
  constexpr int NST = direct_stages(F_BM, BN);
  constexpr int WGN = direct_wave_columns(BN, NW), WGM = NW / WGN;
  constexpr int WTM = F_BM / WGM, WTN = BN / WGN;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must hold whole MFMA tiles");
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int OPA = F_BM * LDS_ROW_U4, OPB = BN * LDS_ROW_U4;  // u4 entries of one operand stage
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  touch_args<(MODE == 0 ? 6 : 8)>(P);
  if (MODE == 0 && P.ncls) touch_args<(int)(sizeof(ClassTab) / 64)>(P.tab);
  DirectWork wk;
  if (!direct_assign<F_BM, BN>(P, block_id, wk)) return;
  const Axis am = wk.am, bn = wk.bn, kax = wk.kax;
  const int m0 = wk.m0, n0 = wk.n0, split = wk.split;
  const int Kn = kax.n;

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int im = 0; im < TM; ++im)
#pragma unroll
    for (int in = 0; in < TN; ++in)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[im][in][v] = 0.0f;

  int li_cb = 0, li_cnt = 0, jn0 = n0, jlim = P.N;  // jn0, jlim: this tile's columns within its block
  if constexpr (MODE == 3) {
    const int tn = n0 / BN;
    li_cb = tn / P.li.tiles;
    jn0 = (tn - li_cb * P.li.tiles) * BN, jlim = P.li.cols;
    li_cnt = imin(imax(P.li.cnt[li_cb], 0), P.li.max);
  }
  // per-tile contraction list (MODE 1): lane l keeps the tile's l-th and (64+l)-th block, a step reads its
  // block out of the lane that holds it, so the loop touches no memory for the list
  int kbl0 = 0, kbl1 = 0;
  bool kb_mode = false;
  if constexpr (MODE == 1) {
    if (P.kb_cnt) {
      kb_mode = true;
      const int* lst = P.kb_list + (long)(n0 / BN) * P.kb_stride;
      const int cnt = Kn >> 6, last = kax.nphys / 64 - 1;
      // (read whatever the count says, from inside the tile's own row of the list: the loads do not wait for it)
      const int e0 = lst[imin(lane, P.kb_stride - 1)], e1 = lst[imin(64 + lane, P.kb_stride - 1)];
      kbl0 = lane < cnt ? imin(imax(e0, 0), last) : 0;
      kbl1 = 64 + lane < cnt ? imin(imax(e1, 0), last) : 0;
    }
  }
  // the channel a row of the tile is stored to, looked up before the contraction instead of after it
  int out_chan = 0;
  if constexpr (MODE == 1) {
    const int i = m0 + tid;
    if (tid < F_BM) out_chan = P.cv.chan && i < P.cv.n_rows ? P.cv.chan[i] : i;
  }
  auto slab = [&](int s, int& ks, int& ksb) {
    if constexpr (MODE == 1) {
      if (kb_mode) {
        ks = (s < 64 ? __builtin_amdgcn_readlane(kbl0, s) : __builtin_amdgcn_readlane(kbl1, s - 64)) * 64;
        const int t = (int)fdiv((uint32_t)ks, P.cv.by_cp), r = (int)fdiv((uint32_t)t, P.cv.by_kw);
        ksb = (r * P.cv.Wg + t - r * P.cv.kw) * P.cv.Cp + (ks - t * P.cv.Cp);
        return;
      }
    }
    direct_slab<MODE>(P, kax, s, ks, ksb);
  };

  if (MODE == 3 ? li_cnt > 0 : Kn > 0) {
    std::conditional_t<MODE == 3, ListLoader<F_BM, NW>, DirectLoader<A_KC, F_BM, NW>> la;
    std::conditional_t<MODE == 3, ListLoader<BN, NW>, DirectLoader<B_KC, BN, NW>> lb;
    const int kbump = MODE == 0 ? direct_kbump(kax) : 0;
    if constexpr (MODE == 3) la.init(P.A, P.lda, am.n, m0, lane, wave);
    else la.init(P.A, P.lda, am, m0, lane, wave, kbump);
    if constexpr (MODE == 3) lb.init_taps(P.B, P.cv, P.li, li_cb, jn0, lane, wave);
    else if constexpr (MODE == 1) lb.init_pixels(P.B, P.cv, n0, lane, wave);
    else if constexpr (MODE == 2) lb.init_tap_columns(P.B, P.cv, P.N, n0, lane, wave);
    else lb.init(P.B, P.ldb, bn, n0, lane, wave, kbump);
    const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)lds);
    // KC: one place per slice, tile i's rows lie 16 i rows further; MC: one per tile, slice q lies 32 q contraction rows further.
    // (an offset has 16 bits: so many stages share their places)
    constexpr int QA = 32 * F_BM * 2, QB = 32 * BN * 2;  // bytes per 32-wide slice of an MC tile
    constexpr int SHARE_A = frag_stages(OPA * 16, A_KC ? (TM - 1) * 2048 : QA + QA / 8), SHARE_B = frag_stages(OPB * 16, B_KC ? (TN - 1) * 2048 : QB + QB / 8);
    constexpr int PA = A_KC ? 2 : TM, PB = B_KC ? 2 : TN;
    unsigned aaddr[(NST + SHARE_A - 1) / SHARE_A][PA], baddr[(NST + SHARE_B - 1) / SHARE_B][PB];
    auto frag_place = [&](int row0, int q) {
      const int row = row0 + (lane & 15);
      return (unsigned)(row * 8 + (((lane >> 4) + 4 * q) ^ kc_swz<false>(row))) * 16u;
    };
#pragma unroll
    for (int i = 0; i * SHARE_A < NST; ++i)
#pragma unroll
      for (int p = 0; p < PA; ++p)
        aaddr[i][p] = lds_base + (unsigned)(i * SHARE_A * OPA) * 16u + (A_KC ? frag_place(wm * WTM, p) : (unsigned)mc_frag_base<F_BM>(wm * WTM + p * 16, lane));
#pragma unroll
    for (int i = 0; i * SHARE_B < NST; ++i)
#pragma unroll
      for (int p = 0; p < PB; ++p)
        baddr[i][p] = lds_base + (unsigned)(NST * OPA + i * SHARE_B * OPB) * 16u + (B_KC ? frag_place(wn * WTN, p) : (unsigned)mc_frag_base<BN>(wn * WTN + p * 16, lane));
    // contraction steps of this workgroup (a share of them when the contraction is split)
    const int S_all = ((MODE == 3 ? li_cnt : Kn) + 63) >> 6;
    const int s_lo = (int)((long)split * S_all / P.splits), s_hi = (int)((long)(split + 1) * S_all / P.splits);
    int S = s_hi - s_lo;
    int* const list = reinterpret_cast<int*>(lds + NST * (OPA + OPB));  // MODE 3: grid pixels of the steps of a chunk
    uint32_t ao[decltype(la)::NI], bo[decltype(lb)::NI];
    auto load_stage = [&](int it, int buf) {
      if constexpr (MODE == 3) {
        la.look(list + it * 64, ao), lb.look(list + it * 64, bo);
#pragma unroll
        for (int j = 0; j < decltype(la)::NI; ++j) la.issue_one(lds + buf * OPA, ao[j], wave, j);
#pragma unroll
        for (int j = 0; j < decltype(lb)::NI; ++j) lb.issue_one(lds + NST * OPA + buf * OPB, bo[j], wave, j);
      } else {
        const int krem = Kn - (s_lo + it) * 64;
        int ks, ksb;
        slab(s_lo + it, ks, ksb);
        const bool tail = krem < 64 || ks + 64 + kbump > kax.nphys;
        if (__builtin_expect(tail, 0)) {
          la.issue_tail(lds + buf * OPA, ks, krem, kax.nphys, lane, wave, kbump);
          lb.issue_tail(lds + NST * OPA + buf * OPB, ksb, krem, MODE == 1 ? 0x7fffffff : kax.nphys, lane, wave, kbump);
        } else {
          la.issue(lds + buf * OPA, ks, wave);
          lb.issue(lds + NST * OPA + buf * OPB, ksb, wave);
        }
      }
    };
    // A step is 2 PARTS units: slice Q of 32 by part H of the wavefront's rows or columns, whichever are more.  The parts share
    // the other operand, so that what two units hold fits beside the accumulators.
    constexpr bool SPLIT_N = TN > TM;
    constexpr int PARTS = TM * TN <= 4 ? 1 : SPLIT_N ? (TN % 7 == 0 ? 7 : 2) : TM * TN >= 32 && TM % 4 == 0 ? 4 : 2;
    constexpr int AF = SPLIT_N ? TM : TM / PARTS, BF = SPLIT_N ? TN / PARTS : TN;
    static_assert((SPLIT_N ? TN : TM) % PARTS == 0, "whole tiles");
    Frag fa[2][AF], fb[2][BF];
    // issue the fragment reads of unit U of stage BUF (compile-time: immediates): the parted operand into set U % 2, the
    // shared one, with a slice's first part, into the slice's set
    auto issue = [&](auto bufc, auto uc) {
      constexpr int BUF = decltype(bufc)::value, U = decltype(uc)::value, Q = U / PARTS, H = U % PARTS;
      constexpr int SA = BUF % SHARE_A * OPA * 16, SB = BUF % SHARE_B * OPB * 16;  // byte offsets of the stage
      if constexpr (SPLIT_N || H == 0) {
        static_for<BF>([&](auto ic) {
          constexpr int I = (SPLIT_N ? H * BF : 0) + decltype(ic)::value;
          Frag& f = fb[SPLIT_N ? U & 1 : Q][decltype(ic)::value];
          if constexpr (B_KC) {
            lds_read_b128<SB + I * 2048>(f.v, baddr[BUF / SHARE_B][Q]);
          } else {
            lds_read_tr16_b64<SB + Q * QB>(f.lo, baddr[BUF / SHARE_B][I]);
            lds_read_tr16_b64<SB + Q * QB + QB / 8>(f.hi, baddr[BUF / SHARE_B][I]);
          }
        });
      }
      if constexpr (!SPLIT_N || H == 0) {
        static_for<AF>([&](auto ic) {
          constexpr int I = (SPLIT_N ? 0 : H * AF) + decltype(ic)::value;
          Frag& f = fa[SPLIT_N ? Q : U & 1][decltype(ic)::value];
          if constexpr (A_KC) {
            lds_read_b128<SA + I * 2048>(f.v, aaddr[BUF / SHARE_A][Q]);
          } else {
            lds_read_tr16_b64<SA + Q * QA>(f.lo, aaddr[BUF / SHARE_A][I]);
            lds_read_tr16_b64<SA + Q * QA + QA / 8>(f.hi, aaddr[BUF / SHARE_A][I]);
          }
        });
      }
    };
    auto wait = [&](int u) {
      const int q = u / PARTS, h = u % PARTS;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (!SPLIT_N || h == 0) {
#pragma unroll
        for (int im = 0; im < AF; ++im) frag_wait<A_KC>(fa[SPLIT_N ? q : u & 1][im]);
      }
      if (SPLIT_N || h == 0) {
#pragma unroll
        for (int in = 0; in < BF; ++in) frag_wait<B_KC>(fb[SPLIT_N ? u & 1 : q][in]);
      }
    };
    // (tiles come out transposed: a lane then holds four neighbouring columns of a row at a time)
    auto mfma = [&](f32x4_t& c, const Frag& x, const Frag& y) {
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_value<B_KC>(y), frag_value<A_KC>(x), c, 0, 0, 0);
    };
    auto mfma_of = [&](int u, int im, int in) {
      const int q = u / PARTS, h = u % PARTS;
      if (SPLIT_N) mfma(acc[im][h * BF + in], fa[q][im], fb[u & 1][in]);
      else mfma(acc[h * AF + im][in], fa[u & 1][im], fb[q][in]);
    };
    // unit U's MFMAs; each(m) runs behind MFMA m of the step, the last unit's being the first (left to itself the scheduler
    // gathers the MFMAs of several units behind their waits)
    constexpr int UNITS = 2 * PARTS, MM = AF * BF;
    auto mma_each = [&](auto uc, auto each) {
      constexpr int U = decltype(uc)::value;
      __builtin_amdgcn_sched_barrier(0);
      static_for<MM>([&](auto ic) {
        constexpr int I = decltype(ic)::value;
        mfma_of(U, I / BF, I % BF);
        each(std::integral_constant<int, (U + 1) % UNITS * MM + I>{});
      });
      __builtin_amdgcn_sched_barrier(0);
    };
    // all units of a stage but the last one's MFMAs; `late` runs behind the others' reads
    auto first_units = [&](auto bufc, auto each, auto late) {
      static_for<UNITS - 1>([&](auto uc) {
        constexpr int U = decltype(uc)::value;
        wait(U);
        issue(bufc, std::integral_constant<int, U + 1>{});
        if constexpr (U == UNITS - 2) late();
        mma_each(uc, each);
      });
      wait(UNITS - 1);
    };
    using I0 = std::integral_constant<int, 0>;
    // The steady loop's slabs come from the iterator (DirectSlabs).
    DirectSlabs<MODE> slabs;
    auto next_slab = [&](int s, int& ks, int& ksb) {
      if constexpr (MODE == 1) {
        if (kb_mode) return slab(s, ks, ksb);
      }
      slabs.next(P, ks, ksb);
    };
    // One contraction step from stage BUF.  A unit's reads are in flight behind the MFMAs of the one before; the stage
    // hand-over (wait for the next stage's loads, barrier, read the next stage's first unit, start the loads of stage it+NST
    // into the buffer just released) sits in front of the LAST unit's MFMAs, so neither the barrier nor the first LDS latency
    // of a stage leaves the matrix cores idle.  Loads complete in order: with NST - 2 younger stages allowed in flight,
    // stage it+1 has landed.
    constexpr int LPS = decltype(la)::NI + decltype(lb)::NI, NA = decltype(la)::NI;  // loads of one thread per stage
    using LastUnit = std::integral_constant<int, UNITS - 1>;
    // Loads go out spread over the MFMAs, from the hand-over on: the memory pipe of a CU takes one in 16 clocks, and a wavefront
    // that finds it full issues no MFMAs either.  Over a step where a stage has two steps to arrive, sooner where it has one.
    constexpr int WINDOW = direct_load_window(F_BM, BN, UNITS * MM, MM);
    int ks = 0, ksb = 0;  // slabs of the stage whose loads are going out
    // loads [LO, HI) of that stage into buffer BUF
    auto loads = [&](auto bufc, auto lo, auto hi) {
      constexpr int BUF = decltype(bufc)::value, LO = decltype(lo)::value;
      static_for<decltype(hi)::value - LO>([&](auto jc) {
        constexpr int L = LO + decltype(jc)::value;
        if constexpr (MODE == 3) {
          if constexpr (L < NA) la.issue_one(lds + BUF * OPA, ao[L], wave, L);
          else lb.issue_one(lds + NST * OPA + BUF * OPB, bo[L - NA], wave, L - NA);
        } else {
          if constexpr (L < NA) la.issue_one(lds + BUF * OPA, ks, wave, L);
          else lb.issue_one(lds + NST * OPA + BUF * OPB, ksb, wave, L - NA);
        }
      });
    };
    constexpr auto loads_before = [](int m) { return (m * LPS + WINDOW - 1) / WINDOW < LPS ? (m * LPS + WINDOW - 1) / WINDOW : LPS; };  // of the window's MFMA m
    auto loads_at = [&](auto bufc, auto mc) {
      constexpr int M = decltype(mc)::value, L0 = loads_before(M), L1 = loads_before(M + 1);
      loads(bufc, std::integral_constant<int, L0>{}, std::integral_constant<int, L1>{});
      if constexpr (L1 > L0) __builtin_amdgcn_sched_barrier(0);
    };
    using LeftOver = std::integral_constant<int, loads_before(MM)>;  // first load that goes out in the step behind the hand-over
    auto step = [&](auto bufc, int it, bool begin_window) {
      constexpr int BUF = decltype(bufc)::value;
      using B = std::integral_constant<int, BUF>;
      using NB = std::integral_constant<int, (BUF + 1) % NST>;
      first_units(B{}, [](auto) {}, [] {});
      if (it + 1 < S) {
        if (it + NST - 1 < S) wait_vmcnt<(NST - 2) * LPS>();
        else wait_vmcnt<0>();
        wg_barrier();  // stage it+1 is complete and visible; nobody reads stage it any more
        issue(NB{}, I0{});
      }
      mma_each(LastUnit{}, [](auto) {});
      // (behind the MFMAs so that nothing but the barrier and one fragment read sits between two units' MFMAs)
      if (begin_window) {
        if constexpr (MODE == 3) la.look(list + (it + NST) * 64, ao), lb.look(list + (it + NST) * 64, bo);
        else next_slab(s_lo + it + NST, ks, ksb);
        loads(B{}, I0{}, LeftOver{});
      } else if (it + NST < S) {
        load_stage(it + NST, BUF);
      }
    };
    // The same step where every question is settled: a successor stage exists, the stage to load
    // exists and is a full one (the axis is affine, or made of whole blocks that hold whole steps:
    // then only the last stage can be partial).  No tail handling, no branches.
    auto steady_step = [&](auto bufc, int it) {
      constexpr int BUF = decltype(bufc)::value;
      using B = std::integral_constant<int, BUF>;
      using NB = std::integral_constant<int, (BUF + 1) % NST>;
      using PB = std::integral_constant<int, (BUF + NST - 1) % NST>;
      first_units(B{}, [&](auto mc) { loads_at(PB{}, mc); }, [&] {
        // (looked up here, the rows of the next loads are known before the loads are issued)
        if constexpr (MODE == 3) la.look(list + (it + NST) * 64, ao), lb.look(list + (it + NST) * 64, bo);
        else next_slab(s_lo + it + NST, ks, ksb);
      });
      wait_vmcnt<(NST - 2) * LPS>();
      wg_barrier();
      issue(NB{}, I0{});
      mma_each(LastUnit{}, [&](auto mc) { loads_at(B{}, mc); });
    };
    auto contract = [&] {
#pragma unroll
      for (int st = 0; st < NST; ++st)
        if (st < S) load_stage(st, st);
      if (S >= NST) wait_vmcnt<(NST - 1) * LPS>();
      else if (NST > 2 && S == 2) wait_vmcnt<LPS>();
      else wait_vmcnt<0>();
      wg_barrier();
      issue(I0{}, I0{});
      // steps it whose stage it+NST is not the last one (only the last can be partial); a window longer than a unit begins in the
      // step before them
      constexpr int LEAD = LeftOver::value < LPS ? 1 : 0;
      const bool steady = (MODE == 3 || direct_full_steps(kax)) && LEAD + 2 * NST < S;
      int it0 = LEAD;
      if (MODE != 3 && steady) slabs.begin(P, kax, s_lo + NST);
      if constexpr (LEAD) step(I0{}, 0, steady);
      if (steady) {
        // (Two words, for where the code behind them lies among the lines of the instruction cache: without them the loop of the
        // 64 x 64 tile begins with the last word of a line, and six dependent launches take 48.8 instead of 48.4 us; begun with a
        // line, those of tile patterns, 128 x 4096 x 4096, took 76.1 instead of 75.2.)
        if constexpr (NW == 4 && (MODE == 0 || MODE == 2)) asm volatile("s_nop 0\n\ts_nop 0");
        for (; it0 + 2 * NST < S; it0 += NST)
          static_for<NST>([&](auto b) { steady_step(std::integral_constant<int, (decltype(b)::value + LEAD) % NST>{}, it0 + decltype(b)::value); });
        if constexpr (LEAD) loads(I0{}, LeftOver{}, std::integral_constant<int, LPS>{});
      }
      for (int it = it0; it < S; it += NST)
        static_for<NST>([&](auto b) {
          if (it + decltype(b)::value < S) step(std::integral_constant<int, (decltype(b)::value + LEAD) % NST>{}, it + decltype(b)::value, false);
        });
    };
    if constexpr (MODE == 3) {
      // as much of this share's list at a time as LDS holds, as pixels of the grid
      constexpr int CAP = direct_list_cap(F_BM);
      const int* src = P.li.list + (long)li_cb * P.li.stride;
      const int top = (int)(P.cv.pix_total - 1);
      for (int e0 = s_lo * 64; e0 < s_hi * 64; e0 += CAP) {
        const int e1 = imin(e0 + CAP, s_hi * 64);
        __syncthreads();
        for (int i = e0 + tid; i < e1; i += 64 * NW) {
          const int p = imin(imax(src[imin(i, li_cnt - 1)], 0), top);
          const int n = (int)fdiv((uint32_t)p, P.cv.per_img), rem = p - n * P.cv.HoWo, ho = (int)fdiv((uint32_t)rem, P.cv.per_row);
          list[i - e0] = i < li_cnt ? n * P.cv.HgWg + ho * P.cv.Wg + rem - ho * P.cv.Wo : P.li.pad;
        }
        __syncthreads();
        S = (e1 - e0) >> 6;
        contract();
      }
    } else if (S > 0) {
      contract();
    }
  }

  // epilogue: lane holds row (lane & 15) of each 16x16 tile, its columns 4*(lane>>4) + v.  The tile goes
  // through LDS (the operand stages are dead once every wave is past its last read) and leaves in 16-byte pieces of its
  // rows.  Straight from the registers, pairs of columns exchanged between lanes to make words, the way out took 18000 of
  // 123000 clocks of a 256 x 256 tile (K = 2048) and 37000 of 86000 of a 256 x 128 tile with fp32 results (K = 1024).
  // With the core of 32 x 32 x 16 MFMAs, before and after: 4096^3 in 64 x 64 tiles at dp = 2 85, 101 and 91 us forward, data and
  // weight gradient, then 79, 94 and 87; projection of 8192 x 1024 -> 2048 to fp32 67, 57 us; 128 x 4096 x 4096 in 32 x 32 tiles at
  // dp = 3, weight gradient 20.8, 17.7 us.
  constexpr int NT = 64 * NW;
  // (the 256 x 256 tile only stores plain results: bf16, and of operands along the contraction fp32)
  constexpr bool GENERAL_OUT = !(F_BM == 256 && BN == 256), WIDE_OUT = GENERAL_OUT || (A_KC && B_KC && MODE == 0);
  // Columns at or beyond the B operand's extent (padding of a compact output) are stored as zeros:
  // the loaders fed them clamped, i.e. arbitrary, rows.
  const int n_valid = (MODE == 0 && P.ncls == 0) ? bn.n : 0x7fffffff;
  char* const tile = reinterpret_cast<char*>(lds);
  // four results at a time, f(row, column, values): columns of the tile
  auto each_quad = [&](auto f) {
#pragma unroll
    for (int im = 0; im < TM; ++im)
#pragma unroll
      for (int in = 0; in < TN; ++in) {
        float x[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = acc[im][in][t];
        f(wm * WTM + im * 16 + (lane & 15), wn * WTN + in * 16 + 4 * (lane >> 4), x);
      }
  };
  auto stage_bf16 = [&] {
    each_quad([&](int r, int c, float (&x)[4]) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        x[t] *= P.alpha;
        if (P.relu) x[t] = fmaxf(x[t], 0.0f);
      }
      *reinterpret_cast<uint2*>(tile + r * direct_pitch(BN, 2) + c * 2) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
    });
  };
  if constexpr (MODE == 1) {
    // NCHW output: compact row i -> channel (through the kept-channel list when there is one), column j -> pixel (n, hw)
    // at n*out_chan*HW + hw; a row of the tile is one run of 2 BN bytes of its channel's plane.
    // N=128, 28x28, 128 -> 256 channels, 3x3: with words of pairs straight from the registers and the channel looked up
    // before each store, a 256 x 256 tile's way out took 20000 of its 81000 clocks, now 9700; the product 82 -> 77 us, the
    // data gradient of 256 channels from 256 (K = 2304) 125 -> 116 us.
    const ConvMap& cv = P.cv;
    const int HW = cv.HoWo;
    constexpr int PITCH = direct_pitch(BN, 2);
    int* const chan = reinterpret_cast<int*>(tile + F_BM * PITCH);
    constexpr int CH = BN / 8;  // 16-byte pieces per row
    constexpr int CL = CH <= 8 ? 8 : CH <= 16 ? 16 : CH <= 32 ? 32 : 64, RS = NT / CL;  // threads along a row, rows at a time
    const int piece = tid % CL, jc = n0 + piece * 8;
    int pix[8];  // of the piece, -1 for padding entries and beyond the last
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const bool in = piece < CH && jc + t < cv.npix;
      pix[t] = in ? (cv.pix ? cv.pix[jc + t] : jc + t) : -1;
    }
    __syncthreads();
    if (tid < F_BM) chan[tid] = out_chan;
    stage_bf16();
    __syncthreads();
    const int r_end = imin(F_BM, cv.n_rows - m0);
    constexpr int U = 4;  // rows at a time: everything read before anything is stored
    if (cv.pix ? !cv.pix_pairs : (HW & 1)) {
      // scattered pixels, or planes that begin at odd places: a lane per pixel
      for (int c0 = 0; c0 < BN; c0 += 64) {
        const int lj = c0 + lane, j = n0 + lj < cv.npix ? (cv.pix ? cv.pix[n0 + lj] : n0 + lj) : -1;
        if (j < 0) continue;
        const int n = (int)fdiv((uint32_t)j, cv.per_img);
        uint16_t* const col = P.C + (long)n * cv.out_chan * HW + (j - n * HW);
        for (int r0 = wave; r0 < r_end; r0 += U * NW) {
          uint16_t v[U];
          int ch[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int r = imin(r0 + u * NW, F_BM - 1);
            ch[u] = chan[r];
            v[u] = *reinterpret_cast<const uint16_t*>(tile + r * PITCH + lj * 2);
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (r0 + u * NW < r_end) col[(long)ch[u] * HW] = v[u];
        }
      }
      return;
    }
    if (piece >= CH) return;
    // Eight pixels that are neighbours in one plane leave as a piece (at any word), pairs as words: planes hold whole words,
    // and listed pixels come in pairs here.
    const bool words = ((uintptr_t)P.C & 3) == 0;
    const int n = (int)fdiv((uint32_t)imax(pix[0], 0), cv.per_img), p0 = pix[0] - n * HW;
    bool whole = pix[0] >= 0 && p0 + 7 < HW && words && (p0 & 1) == 0;
#pragma unroll
    for (int t = 1; t < 8; ++t) whole = whole && pix[t] == pix[0] + t;
    uint16_t* const col = P.C + (long)n * cv.out_chan * HW + p0;
    for (int r0 = tid / CL; r0 < r_end; r0 += U * RS) {
      uint4 v[U];
      int ch[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = imin(r0 + u * RS, F_BM - 1);
        ch[u] = chan[r];
        v[u] = *reinterpret_cast<const uint4*>(tile + r * PITCH + piece * 16);
      }
      if (whole) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (r0 + u * RS < r_end) *reinterpret_cast<U4AnyWord*>(col + (long)ch[u] * HW) = U4AnyWord{v[u].x, v[u].y, v[u].z, v[u].w};
        continue;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int p = pix[2 * t];
        if (p < 0) continue;
        const int np = (int)fdiv((uint32_t)p, cv.per_img);
        uint16_t* const place = P.C + (long)np * cv.out_chan * HW + (p - np * HW);
        const bool word = words && (p & 1) == 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t w = t == 0 ? v[u].x : t == 1 ? v[u].y : t == 2 ? v[u].z : v[u].w;
          if (r0 + u * RS >= r_end) continue;
          uint16_t* const o = place + (long)ch[u] * HW;
          if (word) {
            *reinterpret_cast<uint32_t*>(o) = w;
          } else {
            o[0] = (uint16_t)w;
            if (pix[2 * t + 1] >= 0) o[1] = (uint16_t)(w >> 16);
          }
        }
      }
    }
    return;
  }
  if (GENERAL_OUT && MODE == 0 && P.scatter) {
    // The physical image of as many rows as fit at a time is made in LDS: zeros, then the values at their places, then
    // whole pieces to memory.  (Gathering each piece's elements from a compact tile took 20 thousand clocks of a 64 x 64
    // tile at dp = 2 x 2, eight dependent LDS reads and their index arithmetic per piece.)
    const int sc = P.scn.step, m1 = imin(m0 + F_BM, P.M), n1 = imin(n0 + BN, P.N);
    const int c_lo = n0 * sc, c_hi = n1 == P.N ? P.scn.nphys : n1 * sc;
    // (rows begin an odd number of 16-byte pieces apart: 16 rows at a time start four banks apart)
    const int pitch = ((BN * sc + sc + 14) & ~15) + 8;
    constexpr int LDS_BYTES = (int)direct_lds_bytes(F_BM, BN, 0);
    static_assert(LDS_BYTES / (2 * (((BN * kScatterMaxStep + kScatterMaxStep + 14) & ~15) + 8)) >= 16, "16 rows of the image fit");
    const int rows_fit = imin(F_BM, LDS_BYTES / (pitch * 2) & ~15);
    uint16_t* const img = reinterpret_cast<uint16_t*>(lds);
    for (int r0 = 0; r0 < F_BM && m0 + r0 < m1; r0 += rows_fit) {
      __syncthreads();
      for (int i = tid; i < rows_fit * (pitch >> 3); i += NT) lds[i] = make_uint4(0, 0, 0, 0);
      __syncthreads();
#pragma unroll
      for (int im = 0; im < TM; ++im) {
        const int li = wm * WTM + im * 16 + (lane & 15) - r0, i = m0 + r0 + li;
        if (li < 0 || li >= rows_fit || i >= m1) continue;
        int at = li * pitch + scatter_shift(P, i * P.srm.step + P.srm.off, c_lo) + P.scn.off + (wn * WTN + 4 * (lane >> 4)) * sc;
        // (columns beyond the operand are padding zeros, those beyond the output stay out of the image)
        int nj = imin(n1, n_valid) - (n0 + wn * WTN + 4 * (lane >> 4));
#pragma unroll
        for (int in = 0; in < TN; ++in, at += 16 * sc, nj -= 16) {
          // (opaque: worked out ahead, the places of all columns would take 100 registers, and whether they exist 70 scalar ones)
          asm volatile("" : "+v"(at), "+v"(nj));
          uint16_t* const o = img + at;
#pragma unroll
          for (int t = 0; t < 4; t += 2) {
            float x0 = P.alpha * acc[im][in][t], x1 = P.alpha * acc[im][in][t + 1];
            if (P.relu) x0 = fmaxf(x0, 0.0f), x1 = fmaxf(x1, 0.0f);
            const uint32_t w = pack_bf16x2(x0, x1);
            if (t < nj) o[t * sc] = (uint16_t)w;
            if (t + 1 < nj) o[(t + 1) * sc] = (uint16_t)(w >> 16);
          }
        }
      }
      __syncthreads();
      direct_scatter_rows(lds, pitch, P, m0 + r0, imin(m0 + r0 + rows_fit, m1), c_lo, c_hi, tid, NT);
    }
    return;
  }
  if (MODE == 0 && F_BM * BN <= 64 * 64 && P.part) {
    // Partial sums of a small tile go straight from the registers, 32 bytes of a row at a time: such launches are a few
    // workgroups that are over soon, and the way through LDS took longer (138 x 1152 -> 1664, strides 4 and 8: 6.3 against
    // 5.3 us each for the forward product and the data gradient).
    float* const part = P.part + (long)split * P.M * P.N;
    each_quad([&](int r, int c, float (&x)[4]) {
      const int i = m0 + r, j = n0 + c;
      if (i >= P.M) return;
      float* const o = part + (long)i * P.N + j;
      if (j + 3 < imin(P.N, n_valid)) {
        *reinterpret_cast<U4AnyWord*>(o) = U4AnyWord{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (j + t < P.N) o[t] = j + t < n_valid ? x[t] : 0.0f;
      }
    });
    return;
  }
  // Mapped rows / columns come in blocks that are multiples of 32, so one index lookup per block places all of its rows
  // (columns).
  const bool partial = GENERAL_OUT && P.part;
  const bool wide = WIDE_OUT && (P.part || P.out_f32 || P.beta != 0.0f);  // staged, or stored, as fp32
  constexpr int HALF = F_BM / 2;
  static_assert(HALF * direct_pitch(BN, 4) <= F_BM * direct_pitch(BN, 2) && (size_t)F_BM * (direct_pitch(BN, 2) + 4) <= direct_lds_bytes(F_BM, BN, MODE),
                "either tile ends before the rows' places, and these within the LDS of the launch");
  int* const row_of = reinterpret_cast<int*>(tile + F_BM * direct_pitch(BN, 2));  // physical rows, -1 beyond the output
  __syncthreads();
  if (tid < F_BM) {
    const int i0 = m0 + (tid & ~31), mlim = P.c_rows_mapped ? am.n : P.M, mphys = P.M;
    const int r = partial ? m0 + tid : i0 < mlim ? (P.c_rows_mapped ? ax_phys(am, i0) : i0) + (tid & 31) : mphys;
    row_of[tid] = r < (partial ? P.M : mphys) ? r : -1;
  }
  const int rows = partial || !P.c_rows_mapped ? imin(F_BM, P.M - m0) : F_BM;  // of the tile, that can exist
  constexpr int U = 4;  // rows at a time: everything read before anything is stored
  if (wide) {
    if constexpr (WIDE_OUT) {
      constexpr int PITCH = direct_pitch(BN, 4), CL = BN / 4, RS = NT / CL;
      const int lj = tid % CL * 4, jb = jn0 + lj, j = jb + li_cb * jlim;  // (MODE 3: column within its block, of the product)
      const int nlim = partial ? jlim : P.c_cols_mapped ? bn.n : P.N;
      const int pc = partial ? j : P.c_cols_mapped ? ax_phys(bn, jb & ~31) + (jb & 31) : jb;
      // columns that exist, and that are not padding of a compact output
      const int nc = imin(4, partial ? jlim - jb : P.N - pc), nv = n_valid - jb;
      const long ld = partial ? P.N : P.ldc;
      const float alpha = partial ? 1.0f : P.alpha;
      float* const outf = partial ? P.part + (long)split * P.M * P.N : reinterpret_cast<float*>(P.C);
      const bool relu = !partial && P.relu;
      const bool to_f32 = partial || P.out_f32, general = !partial && (P.beta != 0.0f || P.relu_src || !to_f32);
      // (half of the rows at a time: all of a 128 x 128 tile would take the LDS of the CU's second workgroup)
#pragma unroll 1
      for (int h = 0; h < 2 && h * HALF < rows; ++h) {
        if (h) __syncthreads();
        if (wm / (WGM / 2) == h)
          each_quad([&](int r, int c, float (&x)[4]) { *reinterpret_cast<float4*>(tile + (r - h * HALF) * PITCH + c * 4) = make_float4(x[0], x[1], x[2], x[3]); });
        __syncthreads();
        if (jb >= nlim) continue;
        const int rows_h = imin(HALF, rows - h * HALF);
        if (to_f32 && !general && nc == 4 && nv >= 4) {
          for (int r0 = tid / CL; r0 < rows_h; r0 += U * RS) {
            float4 x[U];
            int pr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const int r = imin(r0 + u * RS, HALF - 1);
              pr[u] = r0 + u * RS < rows_h ? row_of[h * HALF + r] : -1;
              x[u] = *reinterpret_cast<const float4*>(tile + r * PITCH + lj * 4);
              x[u].x *= alpha, x[u].y *= alpha, x[u].z *= alpha, x[u].w *= alpha;
              if (relu) x[u].x = fmaxf(x[u].x, 0.0f), x[u].y = fmaxf(x[u].y, 0.0f), x[u].z = fmaxf(x[u].z, 0.0f), x[u].w = fmaxf(x[u].w, 0.0f);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (pr[u] >= 0)
                *reinterpret_cast<U4AnyWord*>(outf + (long)pr[u] * ld + pc) =
                    U4AnyWord{__float_as_uint(x[u].x), __float_as_uint(x[u].y), __float_as_uint(x[u].z), __float_as_uint(x[u].w)};
          }
          continue;
        }
#pragma unroll 1
        for (int r = tid / CL; r < rows_h; r += RS) {
          const int pr = row_of[h * HALF + r];
          if (pr < 0) continue;
          const float* const q = reinterpret_cast<const float*>(tile + r * PITCH + lj * 4);
          const long at = (long)pr * ld + pc;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            if (t >= nc) break;
            float x = t < nv ? alpha * q[t] : 0.0f;
            if (general && P.beta != 0.0f) x += P.beta * (to_f32 ? outf[at + t] : bf16_bits_to_f32(P.C[at + t]));
            if (relu) x = fmaxf(x, 0.0f);
            if (general && P.relu_src) x = bf16_bits_to_f32(P.relu_src[at + t]) > 0.0f ? x : 0.0f;
            if (to_f32) outf[at + t] = x;
            else P.C[at + t] = f32_to_bf16_bits(x);
          }
        }
      }
    }
    return;
  }
  if constexpr (MODE == 0) {
    constexpr int PITCH = direct_pitch(BN, 2), CL = BN / 8, RS = NT / CL;
    stage_bf16();
    __syncthreads();
    const int nlim = P.c_cols_mapped ? bn.n : P.N, nphys = P.N;
    const uint16_t* const src = GENERAL_OUT ? P.relu_src : nullptr;
    if (((P.ldc & 1) | (int)((uintptr_t)P.C & 3) | (int)((uintptr_t)src & 3)) != 0) {
      // rows that begin at odd places: a lane per column
      for (int c0 = 0; c0 < BN; c0 += 64) {
        const int j = n0 + c0 + lane, pc = j < nlim ? (P.c_cols_mapped ? ax_phys(bn, j & ~31) + (j & 31) : j) : nphys;
        if (pc >= nphys) continue;
        for (int r0 = wave; r0 < rows; r0 += U * NW) {
          uint16_t v[U], g[U];
          int pr[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int r = imin(r0 + u * NW, F_BM - 1);
            pr[u] = r0 + u * NW < rows ? row_of[r] : -1;
            v[u] = j < n_valid ? *reinterpret_cast<const uint16_t*>(tile + r * PITCH + (c0 + lane) * 2) : (uint16_t)0;
          }
          if (src) {
#pragma unroll
            for (int u = 0; u < U; ++u) g[u] = src[(long)imax(pr[u], 0) * P.ldc + pc];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = bf16_bits_to_f32(g[u]) > 0.0f ? v[u] : (uint16_t)0;
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (pr[u] >= 0) P.C[(long)pr[u] * P.ldc + pc] = v[u];
        }
      }
      return;
    }
    const int lj = tid % CL * 8, j = n0 + lj;
    if (j >= nlim) return;
    const int pc = P.c_cols_mapped ? ax_phys(bn, j & ~31) + (j & 31) : j;
    const int nc = imin(8, nphys - pc), nv = n_valid - j;  // columns that exist, that are not padding of a compact output
    if (nc < 8 || nv < 8) {  // the last columns
#pragma unroll 1
      for (int r = tid / CL; r < rows; r += RS) {
        const int pr = row_of[r];
        if (pr < 0) continue;
        const uint16_t* const q = reinterpret_cast<const uint16_t*>(tile + r * PITCH + lj * 2);
        const long at = (long)pr * P.ldc + pc;
#pragma unroll 1
        for (int t = 0; t < nc; ++t) P.C[at + t] = t < nv && (!src || bf16_bits_to_f32(src[at + t]) > 0.0f) ? q[t] : (uint16_t)0;
      }
      return;
    }
    for (int r0 = tid / CL; r0 < rows; r0 += U * RS) {
      uint32_t v[U][4];
      int pr[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = imin(r0 + u * RS, F_BM - 1);
        pr[u] = r0 + u * RS < rows ? row_of[r] : -1;
        const uint4 q = *reinterpret_cast<const uint4*>(tile + r * PITCH + lj * 2);
        v[u][0] = q.x, v[u][1] = q.y, v[u][2] = q.z, v[u][3] = q.w;
      }
      if (src) {
        // ReLU mask of the same positions (same layout as the output)
        uint32_t g[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const U4AnyWord w = *reinterpret_cast<const U4AnyWord*>(src + (long)imax(pr[u], 0) * P.ldc + pc);
          g[u][0] = w.x, g[u][1] = w.y, g[u][2] = w.z, g[u][3] = w.w;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            v[u][t] &= (bf16_bits_to_f32((uint16_t)g[u][t]) > 0.0f ? 0xffffu : 0u) | (bf16_bits_to_f32((uint16_t)(g[u][t] >> 16)) > 0.0f ? 0xffff0000u : 0u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (pr[u] >= 0) *reinterpret_cast<U4AnyWord*>(P.C + (long)pr[u] * P.ldc + pc) = U4AnyWord{v[u][0], v[u][1], v[u][2], v[u][3]};
    }
  }
}

// 16-byte pieces of the dropped tiles, kZeroTileRows rows of the matrix per workgroup.  In the product's launch because
// the two write different places: as a launch before it, the zeros of a 4096 x 4096 gradient took 10 us of their own.
constexpr int kZeroTileRows = 8;
template <int NT> __device__ __forceinline__ void zero_tiles_body(const ZeroTilesJob& z, uint16_t* C, int ld, int block) {
  const int chunks = z.cols >> 3, r0 = block * kZeroTileRows, n = imin(kZeroTileRows, z.rows - r0) * chunks;
  for (int i = threadIdx.x; i < n; i += NT) {
    const int r = (int)fdiv((uint32_t)i, z.by_chunks), c = i - r * chunks;
    const int t = (int)fdiv((uint32_t)(r0 + r), z.by_tr) * z.TC + (int)fdiv((uint32_t)c, z.by_tc);
    if ((t + z.dp - z.o) % z.dp) *reinterpret_cast<uint4*>(C + (long)(r0 + r) * ld + c * 8) = make_uint4(0, 0, 0, 0);
  }
}

// (wavefronts per SIMD: as many workgroups as their LDS lets share a CU)
template <bool A_KC, bool B_KC, int F_BM, int BN, int NW, int MODE = 0>
__global__ __launch_bounds__(64 * NW, F_BM + BN <= 192 ? 3 : 2) void gemm_direct_kernel(const FastParams P) {
  extern __shared__ uint4 direct_lds[];
  if constexpr (MODE == 0 && !A_KC && !B_KC) {
    const int z = (int)blockIdx.x - ((int)gridDim.x - P.zt.blocks);
    if (z >= 0) return zero_tiles_body<64 * NW>(P.zt, P.C, P.ldc, z);
  }
  direct_body<A_KC, B_KC, F_BM, BN, NW, MODE>(P, (int)blockIdx.x, direct_lds);
}

// Finishing pass of a product whose result could not be stored by the GEMM itself (split
// contraction, or an output scattered at element granularity with dropped positions to zero):
// sums the fp32 partials part[split][M][N] and writes the output through its maps, walking the
// PHYSICAL output when dropped positions have to be written.
__device__ __forceinline__ int ax_inverse(const Axis& a, int p) {
  // compact index of physical index p, or -1
  if (a.kind == AX_AFFINE) {
    const int d = p - a.off;
    if (d < 0 || d % a.step) return -1;
    const int j = d / a.step;
    return j < a.n ? j : -1;
  }
  if (a.kind == AX_LIST) {
    int lo = 0, hi = a.n - 1;
    while (lo <= hi) {
      const int mid = (lo + hi) >> 1, v = a.list[mid];
      if (v == p) return mid;
      if (v < p) lo = mid + 1;
      else hi = mid - 1;
    }
    return -1;
  }
  return -1;
}

template <typename T>
__global__ __launch_bounds__(256) void gemm_finish_kernel(const float* part, int splits, int M, int N, OutMat C) {
  const int rows = C.fill ? C.rm.nphys : M, cols = C.fill ? C.cn.nphys : N;
  const long total = (long)rows * cols;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const int r = (int)(e / cols), c = (int)(e - (long)r * cols);
    int i, j, pr, pc;
    if (C.fill) {
      pr = r, pc = c;
      i = ax_inverse(C.rm, r);
      j = ax_inverse(C.cn, c);
    } else {
      i = r, j = c;
      pr = ax_phys(C.rm, r);
      pc = ax_phys(C.cn, c);
    }
    float x = 0.0f;
    if (i >= 0 && j >= 0) {
      const float* p = part + (long)i * N + j;
      for (int s = 0; s < splits; ++s) x += p[(long)s * M * N];
      x *= C.alpha;
    }
    store_out<T>(C, (long)pr * C.ld + pc, x, true);
  }
}

// The same pass for bf16 outputs whose rows can be written in 16-byte pieces (host checks:
// bf16 result, beta == 0, 16-byte aligned rows, column count a multiple of 8; without zero
// fill the column map is the identity).  A thread produces 8 adjacent physical columns.
struct FinishArgs {
  const float* part;
  int splits, M, N;
  OutMat C;
};
static __device__ __forceinline__ void finish_vec_body(const FinishArgs& a, const int bx, const int by, const int gy) {
  const float* part = a.part;
  const int splits = a.splits, M = a.M, N = a.N;
  const OutMat& C = a.C;
  // grid: x over the 8-column pieces of a row, y over rows (uniform per workgroup, so the row
  // lookup is scalar work)
  const int rows = C.fill ? C.rm.nphys : M, cols8 = (C.fill ? C.cn.nphys : N) >> 3;
  const long MN = (long)M * N;
  const int piece = bx * 256 + threadIdx.x;
  if (piece >= cols8) return;
  const int c0 = piece * 8;
  // Workgroup ids go round-robin over the 8 XCDs: XCD x takes the contiguous rows
  // [x * chunk, (x + 1) * chunk).  (Row r on XCD r % 8 would put every kept row of a step-8
  // pattern, i.e. all the work, on one XCD.)
  const int chunk = (rows + 7) >> 3;
  for (int y = by; y < chunk * 8; y += gy) {
    const int r = (y & 7) * chunk + (y >> 3);
    if (r >= rows) continue;
    const int i = C.fill ? ax_inverse(C.rm, r) : r;
    const int pr = C.fill ? r : ax_phys(C.rm, r);
    const long idx = (long)pr * C.ld + c0;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (i >= 0) {
      uint4 gate = make_uint4(0, 0, 0, 0);
      if (C.relu_src) gate = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(C.relu_src) + idx);
      const uint32_t* gw = reinterpret_cast<const uint32_t*>(&gate);
      int j = C.fill ? -1 : c0;
      if (C.fill && C.cn.kind == AX_AFFINE) {
        // first kept column at or after c0 (exact for the 24-bit operands of this division)
        const int d = c0 - C.cn.off + C.cn.step - 1;
        j = 0;
        if (d >= C.cn.step) {
          j = (int)((float)d / (float)C.cn.step);
          j += ((j + 1) * C.cn.step <= d) - (j * C.cn.step > d);
        }
      }
      int jj[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (!C.fill) jj[t] = j + t;
        else if (C.cn.kind == AX_AFFINE) jj[t] = (j < C.cn.n && C.cn.off + j * C.cn.step == c0 + t) ? j++ : -1;
        else jj[t] = ax_inverse(C.cn, c0 + t);
      }
      // The 8 loads of one split are independent and unconditional (positions that are not kept read some kept one
      // and are masked out: behind branches every load would be waited for by itself); splits are summed in order.
      float x[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
      const float* prow = part + (long)i * N;
      uint32_t keep[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        keep[t] = jj[t] >= 0 ? ~0u : 0u;
        asm("" : "+v"(keep[t]));
        jj[t] = imax(jj[t], 0);
      }
      for (int sp = 0; sp < splits; ++sp) {
        float v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = prow[sp * MN + jj[t]];
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] += v[t];
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float v = x[t] * C.alpha;
        if (C.relu) v = fmaxf(v, 0.0f);
        if (C.relu_src) {
          const uint32_t g = (gw[t >> 1] >> (16 * (t & 1))) & 0xffffu;
          v = bf16_bits_to_f32((uint16_t)g) > 0.0f ? v : 0.0f;
        }
        w[t >> 1] |= ((uint32_t)f32_to_bf16_bits(v) & keep[t]) << (16 * (t & 1));
      }
    }
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(C.p) + idx) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

static __global__ __launch_bounds__(256) void gemm_finish_vec_kernel(const FinishArgs a) {
  finish_vec_body(a, (int)blockIdx.x, (int)blockIdx.y, (int)gridDim.y);
}

// Rows of a bf16 matrix that an affine row map (off + i * step, i < n_kept) does NOT reach, set to +0.0:
// the dropped output neurons of a weight gradient.  Independent of the product that writes the kept rows.
struct ZeroRowsArgs {
  uint16_t* C;
  int ld, rows, cols, off, step, n_kept, vec;
};
static __device__ __forceinline__ void zero_rows_body(const ZeroRowsArgs& a, const int bx, const int nblocks) {
  const int dropped = a.rows - a.n_kept;
  // pieces of 16 bytes, of every row's own alignment where rows are no whole number of them
  const int per_row = a.vec ? a.cols >> 3 : (a.cols + 14) >> 3;
  const long total = (long)dropped * per_row;
  for (long e = (long)bx * 256 + threadIdx.x; e < total; e += (long)nblocks * 256) {
    // (a 64-bit division costs several times a 32-bit one, and nearly every matrix stays below 2^32 pieces)
    const int d = total < (1L << 32) ? (int)((uint32_t)e / (uint32_t)per_row) : (int)(e / per_row);
    const int c = (int)(e - (long)d * per_row);
    // d-th dropped row: rows before `off` come first, then step - 1 per group, then the tail
    int r;
    if (d < a.off) {
      r = d;
    } else {
      const int q = (d - a.off) / (a.step - 1), t = (d - a.off) - q * (a.step - 1);
      r = q < a.n_kept ? a.off + q * a.step + 1 + t : a.off + a.n_kept * a.step + (d - a.off - a.n_kept * (a.step - 1)) - (a.step - 1);
    }
    uint16_t* rowp = a.C + (long)r * a.ld;
    const int c0 = c * 8 - (a.vec ? 0 : (int)((reinterpret_cast<uintptr_t>(rowp) & 15) >> 1));
    if (c0 >= 0 && c0 + 8 <= a.cols) {
      *reinterpret_cast<uint4*>(rowp + c0) = make_uint4(0, 0, 0, 0);
    } else {
      for (int q = imax(c0, 0); q < c0 + 8 && q < a.cols; ++q) rowp[q] = 0;
    }
  }
}
static __global__ __launch_bounds__(256) void zero_rows_kernel(const ZeroRowsArgs a) {
  zero_rows_body(a, (int)blockIdx.x, (int)gridDim.x);
}

// Zero the dropped tiles of a tile-masked matrix (weight gradient): one workgroup per tile.
template <typename T>
static __global__ __launch_bounds__(256) void zero_dropped_tiles_kernel(T* C, int ld, int rows, int cols, int tr, int tc,
                                                                 int TC, int dp, int o) {
  const int t = blockIdx.x;
  if (((t + dp - o) % dp) == 0) return;  // kept tile: written by the GEMM
  const int r0 = (t / TC) * tr, c0 = (t % TC) * tc;
  const int h = min(tr, rows - r0), w = min(tc, cols - c0);
  constexpr int CE = ElemTraits<T>::CE;
  if (((w | c0 | ld) & (CE - 1)) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0) {
    const int w8 = w / CE;
    for (int i = threadIdx.x; i < h * w8; i += 256) {
      const int r = i / w8, c = (i - r * w8) * CE;
      *reinterpret_cast<uint4*>(C + (long)(r0 + r) * ld + c0 + c) = make_uint4(0, 0, 0, 0);
    }
  } else {
    for (int i = threadIdx.x; i < h * w; i += 256) {
      const int r = i / w, c = i - r * w;
      C[(long)(r0 + r) * ld + c0 + c] = 0;
    }
  }
}

// an XCD's share should be about square in tiles: bands of group_m tile rows
static inline int direct_group_m(int total_tiles) {
  const int per_xcd = ceil_div(total_tiles, 8);
  int gm = 1;
  while (gm * gm * 2 <= per_xcd && gm < 8) gm *= 2;
  return gm;
}
template <class Params> static inline void set_bands(Params& P, int group_m) {
  P.ncls = P.tab.ncls;
  P.group_m = group_m;
  P.tiles_div = fast_div((uint32_t)imax(P.total_tiles, 1)), P.band_div = fast_div((uint32_t)imax(group_m * P.tiles_n, 1));
}

// Classes of a tile pattern (tiles of x by y, every dp-th from tile o on, over a TR x TC grid of W[O x I]) for
// op 0: Y = X . W^T, 1: dX = dY . W, 2: dW = dY^T . X.  Fills everything but the workgroup counts; false: more
// classes than the table holds.
static inline bool tile_classes(int op, int O, int I, int TR, int TC, int x, int y, int dp, int o, ClassTab& t) {
  int a = TC, b = dp;
  while (b) {
    const int r = a % b;
    a = b;
    b = r;
  }
  const int Pp = dp / a;  // a = gcd(TC, dp)
  if (Pp > F_MAXCLS || (op == 1 && dp > F_MAXCLS)) return false;
  auto cnt = [](int total, int first, int step) { return first < total ? (total - first + step - 1) / step : 0; };
  auto first_col = [&](int c) { return (int)((((long)o - (long)c * TC) % dp + dp) % dp); };
  if (op == 1) {
    t.ncls = dp;
    t.n_step = dp, t.n_bs = y, t.n_phys = I;
    t.k_step = Pp, t.k_bs = x, t.k_phys = O;
    for (int c = 0; c < dp; ++c) {
      t.n_off[c] = c;
      t.n_cnt[c] = cnt(TC, c, dp);
      int J0 = -1;
      for (int J = 0; J < Pp && J0 < 0; ++J)
        if ((((long)J * TC + c - o) % dp + dp) % dp == 0) J0 = J;
      t.k_off[c] = J0 < 0 ? 0 : J0;
      t.k_cnt[c] = J0 < 0 ? 0 : cnt(TR, J0, Pp);
    }
    return true;
  }
  t.ncls = Pp;
  if (op == 0) {
    t.n_step = Pp, t.n_bs = x, t.n_phys = O;
    t.k_step = dp, t.k_bs = y, t.k_phys = I;
    for (int c = 0; c < Pp; ++c) {
      t.n_off[c] = c;
      t.n_cnt[c] = cnt(TR, c, Pp);
      t.k_off[c] = first_col(c);
      t.k_cnt[c] = cnt(TC, t.k_off[c], dp);
    }
  } else {
    t.m_step = Pp, t.m_bs = x, t.m_phys = O;
    t.n_step = dp, t.n_bs = y, t.n_phys = I;
    for (int c = 0; c < Pp; ++c) {
      t.m_off[c] = c;
      t.m_cnt[c] = cnt(TR, c, Pp);
      t.n_off[c] = first_col(c);
      t.n_cnt[c] = cnt(TC, t.n_off[c], dp);
    }
  }
  return true;
}
// Workgroups per class for BM x BN tiles over B rows (op 2: over the class's own rows); `heavy` ones have
// something to contract.  Returns their total.
static inline int count_classes(int op, ClassTab& t, int B, int bm, int bn, int& heavy) {
  auto runs = [](int cnt, int bs, int w) { return bs <= w ? ceil_div(cnt, w / bs) : cnt * (bs / w); };
  int total = 0;
  heavy = 0;
  for (int c = 0; c < t.ncls; ++c) {
    const int mb = op == 2 ? runs(t.m_cnt[c], t.m_bs, bm) : ceil_div(B, bm), nb = runs(t.n_cnt[c], t.n_bs, bn);
    t.mblk[c] = mb > 0 ? mb : 1;
    t.nblk[c] = mb > 0 ? mb * nb : 0;
    total += t.nblk[c];
    if (op == 2 || t.k_cnt[c] > 0) heavy += t.nblk[c];
  }
  return total;
}
static inline bool tile_run_fits(int bs, int w) { return bs <= w ? w % bs == 0 : bs % w == 0; }

// Grid of a plain (class-free) launch: every XCD takes the share [x*n/8, (x+1)*n/8) of the tiles.
static inline int direct_plain_grid(int total_tiles) {
  int worst = 0;
  for (int x = 0; x < 8; ++x) {
    const int sum = (int)((long)(x + 1) * total_tiles / 8) - (int)((long)x * total_tiles / 8);
    worst = sum > worst ? sum : worst;
  }
  return worst * 8;
}

// Grid of a class launch: every XCD takes the share [x*n/8, (x+1)*n/8) of each class.
static inline int class_grid(const ClassTab& t) {
  int worst = 0;
  for (int x = 0; x < 8; ++x) {
    int sum = 0;
    for (int c = 0; c < t.ncls; ++c) sum += (int)((long)(x + 1) * t.nblk[c] / 8) - (int)((long)x * t.nblk[c] / 8);
    worst = sum > worst ? sum : worst;
  }
  return worst * 8;
}

// ---- host-side bounds proof of the LDS-direct loaders -------------------------------------------
// A lane of these kernels forms its global address as base + uniform slab offset + per-lane offset
// with no bounds test in the loop, so the host shows before every launch that no lane of any
// workgroup can leave the operand (a_elems / b_elems elements behind A / B, stated by the caller).
//  * direct_envelope (always, O(classes)): the extreme physical rows, columns and contraction
//    indices the clamps in DirectLoader::init* and the tail rules allow, as inequalities.
//  * direct_prove (dry-run mode and ARD_PROVE_BOUNDS=1, every workgroup x wave x lane x step): runs
//    the kernel's own assignment and address arithmetic (direct_assign, DirectLoader::init*,
//    direct_slab, tail_live are host-callable) and records the smallest and largest byte touched;
//    the steady loop's iterator (DirectSlabs) is stepped beside direct_slab and has to give the same slabs.
static inline bool axis_rows_ok(const Axis& r, bool has_list) {
  // rows of a KC operand after the clamp of init(): min(row, n-1), block axes also clamped to nphys-1
  if (r.n < 1 || r.nphys < 1) return false;
  if (r.kind == AX_AFFINE) return r.off >= 0 && r.step >= 0 && (long)r.off + (long)(r.n - 1) * r.step < r.nphys;
  if (r.kind == AX_BAFF) return r.off >= 0 && r.step >= 0 && r.bs >= 1;
  if (r.kind == AX_LIST) return has_list && r.n <= r.nphys;  // entries are the caller's contract
  return false;
}
static inline bool axis_cols_ok(const Axis& r, int ld) {
  // 8-column runs of an MC operand after the clamp of init(): min(col, n-8), block axes to nphys-8
  if (r.n < 8 || r.nphys < 8 || r.nphys > ld) return false;
  if (r.kind == AX_AFFINE) return r.step == 1 && r.off >= 0 && r.off + r.n <= r.nphys;
  if (r.kind == AX_BAFF) return r.off >= 0 && r.step >= 0 && r.bs >= 8 && (r.bs % 8) == 0;
  return false;
}

template <bool A_KC, bool B_KC, int BM, int BN, int MODE>
static int32_t direct_envelope(const FastParams& F) {
  if (F.a_elems <= 0 || F.b_elems <= 0) return fail(ARD_EINVAL, "bounds proof: operand extents not stated");
  if (F.a_elems >= (1L << 31) || F.b_elems >= (1L << 31)) return fail(ARD_ESHAPE, "bounds proof: operand beyond 32-bit offsets");
  if (F.lda < 8 || F.ldb < 8) return fail(ARD_ESHAPE, "bounds proof: leading dimension below one 16-byte run");
  if constexpr (MODE == 3) {
    // every list entry is clamped to a pixel of the grid, the filler included; columns are clamped to the axis
    const ConvMap& cv = F.cv;
    const ListMap& l = F.li;
    if (!l.list || !l.cnt || l.tiles < 1 || l.cols < 8 || l.cols_per_tap < 8 || (l.cols_per_tap % 8) || (l.chans % 8) || l.max > l.stride || F.am.n < 8)
      return fail(ARD_EINVAL, "bounds proof: bad position list");
    if (cv.pix_total < 1 || cv.Cp < 64 || (cv.Cp % 64) || cv.kw < 1 || F.lda % 64) return fail(ARD_ESHAPE, "bounds proof: bad grid");
    const int row = cv.pix_total - 1, n = row / cv.HoWo, rem = row - n * cv.HoWo;
    const long at = (long)n * cv.HgWg + (long)(rem / cv.Wo) * cv.Wg + rem % cv.Wo, last = at > l.pad ? at : l.pad;
    const int tl = (l.cols - 8) / l.cols_per_tap, cbs = F.tiles_n / l.tiles;
    const long shift = (long)(tl / cv.kw) * cv.Wg + tl % cv.kw;
    if (l.pad < 0 || last >= (1L << 24) || (last + 1) * F.lda > F.a_elems || F.am.n > F.lda || (last + shift + 1) * cv.Cp > F.b_elems ||
        (long)(cbs - 1) * l.chans + l.cols_per_tap > cv.Cp)
      return fail(ARD_ESHAPE, "bounds proof: listed pixels leave the grid");
    return ARD_OK;
  }
  const ClassTab& t = F.tab;
  const int ncls = t.ncls ? t.ncls : 1;
  for (int c = 0; c < ncls; ++c) {
    if (t.ncls && t.nblk[c] == 0) continue;
    // the maps a workgroup of this class can get (direct_assign): whole progression of the class
    Axis am = F.am, bn = F.bn, k = F.k;
    if (t.ncls) {
      if (t.m_bs) am = axis_baff(t.m_off[c], t.m_step, t.m_bs, t.m_cnt[c], t.m_phys);
      bn = axis_baff(t.n_off[c], t.n_step, t.n_bs, t.n_cnt[c], t.n_phys);
      if (t.k_bs) k = axis_baff(t.k_off[c], t.k_step, t.k_bs, t.k_cnt[c], t.k_phys);
    }
    if (k.n <= 0) continue;  // nothing is loaded
    if (k.kind != AX_AFFINE && k.kind != AX_BAFF) return fail(ARD_EINVAL, "bounds proof: contraction map kind %d", k.kind);
    if (k.kind == AX_AFFINE && (k.step != 1 || k.off < 0 || k.off + k.n > k.nphys))
      return fail(ARD_ESHAPE, "bounds proof: contraction [%d, %d) outside its extent %d", k.off, k.off + k.n, k.nphys);
    if (k.kind == AX_BAFF && (k.off < 0 || k.step < 0 || k.bs < 32 || (k.bs % 64 && k.bs != 32)))
      return fail(ARD_ESHAPE, "bounds proof: contraction blocks of %d", k.bs);
    // 32-wide blocks: the upper half of a step lies `step` blocks further; the last kept block must
    // start inside the extent (a step that reaches beyond it takes the tail rule, chunk by chunk)
    if (k.kind == AX_BAFF && k.bs == 32 &&
        ((k.nphys % 8) || (k.n % 32) || ((long)k.off + (long)(k.n / 32 - 1) * k.step) * 32 >= k.nphys))
      return fail(ARD_ESHAPE, "bounds proof: 32-wide contraction blocks (%d of them from %d every %d) leave the extent %d", k.n / 32,
                  k.off, k.step, k.nphys);
    // every contraction index a live lane touches is < k.nphys (full steps need ks + 64 <= nphys, the
    // lanes of a partial step test their own chunk against nphys)
    const long kphys = k.nphys;
    // A
    if (A_KC) {
      if (!axis_rows_ok(am, F.A != nullptr) || kphys > F.lda || (long)am.nphys * F.lda > F.a_elems)
        return fail(ARD_ESHAPE, "bounds proof: A rows (kind %d, n %d, extent %d, ld %d, k %ld) leave %ld elements", am.kind, am.n,
                    am.nphys, F.lda, kphys, F.a_elems);
    } else {
      if (!axis_cols_ok(am, F.lda) || kphys * F.lda > F.a_elems)
        return fail(ARD_ESHAPE, "bounds proof: A columns (kind %d, n %d, extent %d, ld %d, k %ld) leave %ld elements", am.kind,
                    am.n, am.nphys, F.lda, kphys, F.a_elems);
    }
    // B
    if (MODE == 1) {
      const ConvMap& cv = F.cv;
      if (cv.npix < 1 || cv.Cp < 64 || (cv.Cp % 64) || cv.kw < 1 || kphys % cv.Cp) return fail(ARD_ESHAPE, "bounds proof: bad grid");
      // (a list with per-tile contraction lists is padded tile by tile and may be longer than the pixels)
      if (cv.pix && (cv.pix_total < 1 || (cv.npix > cv.pix_total && !F.kb_cnt)))
        return fail(ARD_ESHAPE, "bounds proof: pixel list longer than the pixels");
      if (F.kb_cnt && (!cv.pix || !F.kb_list || F.kb_stride < 1 || F.splits > 1 || k.kind != AX_AFFINE || (kphys % 64)))
        return fail(ARD_EINVAL, "bounds proof: per-tile contraction lists need a pixel list, whole 64-wide blocks and no split");
      const int row = (cv.pix ? cv.pix_total : cv.npix) - 1, n = row / cv.HoWo, rem = row - n * cv.HoWo;
      const long base = (long)n * cv.HgWg + (long)(rem / cv.Wo) * cv.Wg + rem % cv.Wo;
      const int tl = (int)(kphys / cv.Cp) - 1;  // last tap
      const long last = base + (long)(tl / cv.kw) * cv.Wg + tl % cv.kw;
      if ((last + 1) * cv.Cp > F.b_elems) return fail(ARD_ESHAPE, "bounds proof: patch rows leave the grid");
    } else if (MODE == 2) {
      const ConvMap& cv = F.cv;
      if (F.N < 8 || cv.Cp < 64 || (cv.Cp % 64) || cv.kw < 1) return fail(ARD_ESHAPE, "bounds proof: bad grid");
      const int tl = (F.N - 8) / cv.Cp;
      const long shift = (long)(tl / cv.kw) * cv.Wg + tl % cv.kw;
      if ((kphys - 1 + shift + 1) * cv.Cp > F.b_elems) return fail(ARD_ESHAPE, "bounds proof: shifted grid rows leave the grid");
    } else if (B_KC) {
      if (!axis_rows_ok(bn, F.B != nullptr) || kphys > F.ldb || (long)bn.nphys * F.ldb > F.b_elems)
        return fail(ARD_ESHAPE, "bounds proof: B rows (kind %d, n %d, extent %d, ld %d, k %ld) leave %ld elements", bn.kind, bn.n,
                    bn.nphys, F.ldb, kphys, F.b_elems);
    } else {
      if (!axis_cols_ok(bn, F.ldb) || kphys * F.ldb > F.b_elems)
        return fail(ARD_ESHAPE, "bounds proof: B columns (kind %d, n %d, extent %d, ld %d, k %ld) leave %ld elements", bn.kind,
                    bn.n, bn.nphys, F.ldb, kphys, F.b_elems);
    }
  }
  return ARD_OK;
}

// A LIST axis cannot be read on the host: its two extreme readings (every row first / last) bound it.
static inline Axis axis_list_surrogate(const Axis& r, bool last) {
  return r.kind == AX_LIST ? Axis{nullptr, AX_AFFINE, last ? r.nphys - 1 : 0, 0, 1, r.n, r.nphys} : r;
}

template <bool A_KC, bool B_KC, int BM, int BN, int NW, int MODE>
static int32_t direct_prove(const FastParams& P_in, int grid_x, DirectBounds& out) {
  constexpr long NONE_LO = 0x7fffffffffffffffL;
  out = DirectBounds{NONE_LO, -1, NONE_LO, -1, 0};
  using LA = DirectLoader<A_KC, BM, NW>;
  using LB = DirectLoader<B_KC, BN, NW>;
  FastParams P = P_in;
  P.kb_cnt = nullptr;  // device memory: every list of whole blocks stays inside the full contraction walked here
  P.kb_list = nullptr;
  for (int bid = 0; bid < grid_x; ++bid) {
    DirectWork wk;
    if (!direct_assign<BM, BN>(P, bid, wk)) continue;
    const int Kn = wk.kax.n;
    if (Kn <= 0) continue;
    const int S_all = (Kn + 63) >> 6;
    const int s_lo = (int)((long)wk.split * S_all / P.splits), s_hi = (int)((long)(wk.split + 1) * S_all / P.splits);
    if (direct_full_steps(wk.kax)) {
      DirectSlabs<MODE> it;
      const int s0 = s_lo + direct_stages(BM, BN);
      if (s0 < s_hi) it.begin(P, wk.kax, s0);
      for (int s = s0; s < s_hi; ++s) {
        int ks, ksb, is, isb;
        direct_slab<MODE>(P, wk.kax, s, ks, ksb);
        it.next(P, is, isb);
        if (is != ks || isb != ksb) return fail(ARD_ESHAPE, "bounds proof: step %d at %d, %d and not at %d, %d", s, is, isb, ks, ksb);
      }
      if (s0 < s_hi) out.slabs += s_hi - s0;
    }
    for (int pass = 0; pass < 2; ++pass) {  // (second pass only differs for LIST axes and pixel lists)
      if (pass == 1 && wk.am.kind != AX_LIST && wk.bn.kind != AX_LIST && !P.cv.pix) break;
      const Axis am = axis_list_surrogate(wk.am, pass == 1), bn = axis_list_surrogate(wk.bn, pass == 1);
      ConvMap cvp = P.cv;  // a pixel list lives in device memory: its two extreme readings bound it
      if (cvp.pix) cvp.pix = nullptr, cvp.pix_fixed = pass == 1 ? cvp.pix_total - 1 : 0;
      for (int wave = 0; wave < NW; ++wave)
        for (int lane = 0; lane < 64; ++lane) {
          LA la;
          LB lb;
          const int kbump = MODE == 0 ? direct_kbump(wk.kax) : 0;
          la.init(P.A, P.lda, am, wk.m0, lane, wave, kbump);
          if constexpr (MODE == 1) lb.init_pixels(P.B, cvp, wk.n0, lane, wave);
          else if constexpr (MODE == 2) lb.init_tap_columns(P.B, P.cv, P.N, wk.n0, lane, wave);
          else lb.init(P.B, P.ldb, bn, wk.n0, lane, wave, kbump);
          for (int s = s_lo; s < s_hi; ++s) {
            const int krem = Kn - s * 64;
            int ks, ksb;
            direct_slab<MODE>(P, wk.kax, s, ks, ksb);
            const bool tail = krem < 64 || ks + 64 + kbump > wk.kax.nphys;
            const int kend_b = MODE == 1 ? 0x7fffffff : wk.kax.nphys;
            for (int j = 0; j < LA::NI; ++j) {
              if (tail && !LA::tail_live(lane, wave, j, ks, krem, wk.kax.nphys, kbump)) continue;
              const long o = la.byte_offset(j, ks);
              out.a_lo = o < out.a_lo ? o : out.a_lo;
              out.a_hi = o + 16 > out.a_hi ? o + 16 : out.a_hi;
            }
            for (int j = 0; j < LB::NI; ++j) {
              if (tail && !LB::tail_live(lane, wave, j, ksb, krem, kend_b, kbump)) continue;
              const long o = lb.byte_offset(j, ksb);
              out.b_lo = o < out.b_lo ? o : out.b_lo;
              out.b_hi = o + 16 > out.b_hi ? o + 16 : out.b_hi;
            }
          }
        }
    }
  }
  const long a_bytes = (P.a_elems - extent_slack()) * 2, b_bytes = (P.b_elems - extent_slack()) * 2;
  if (out.a_hi >= 0 && (out.a_lo < 0 || out.a_hi > a_bytes))
    return fail(ARD_ESHAPE, "bounds proof: A bytes [%ld, %ld) outside [0, %ld)", out.a_lo, out.a_hi, a_bytes);
  if (out.b_hi >= 0 && (out.b_lo < 0 || out.b_hi > b_bytes))
    return fail(ARD_ESHAPE, "bounds proof: B bytes [%ld, %ld) outside [0, %ld)", out.b_lo, out.b_hi, b_bytes);
  return ARD_OK;
}

// Kinds of LDS-direct products the grouped kernel holds (the 4-wavefront tiles a batch-1024 layer chain
// uses); -1: this instantiation is always launched by itself.
enum { GK_DIRECT_KK_64 = 0, GK_DIRECT_KM_64 = 1, GK_DIRECT_MM_64 = 2, GK_DIRECT_MM_128x64 = 3, GK_COMPACT_W = 10, GK_FINISH_VEC = 11,
       GK_ZERO_ROWS = 12 };
template <bool A_KC, bool B_KC, int BM, int BN, int NW, int MODE>
constexpr int direct_group_kind() {
  if (MODE != 0 || NW != 4) return -1;
  if (BM == 64 && BN == 64) return A_KC ? (B_KC ? GK_DIRECT_KK_64 : GK_DIRECT_KM_64) : (B_KC ? -1 : GK_DIRECT_MM_64);
  if (BM == 128 && BN == 64 && !A_KC && !B_KC) return GK_DIRECT_MM_128x64;
  return -1;
}
// records the launch in this thread's open batch; false: no batch is open (gemm.hip)
bool batch_push_direct(int kind, const FastParams& F, int grid_x, size_t lds_bytes);
bool batch_push_finish(const FinishArgs& a, int gx, int gy);
bool batch_push_zero_rows(const ZeroRowsArgs& a, int gx);

// Host side: launch one instantiation with its dynamic LDS (stages x (BM + BN) rows of 128 bytes);
// kernels above the 64 KiB default get their limit raised once.
template <bool A_KC, bool B_KC, int BM, int BN, int NW, int MODE>
static int32_t launch_direct_alone(const FastParams& F, int grid_x, hipStream_t stream) {
  auto kernel = gemm_direct_kernel<A_KC, B_KC, BM, BN, NW, MODE>;
  const size_t lds_bytes = direct_lds_bytes(BM, BN, MODE);
  static thread_local bool raised = false;
  if (!raised && lds_bytes >= 65536) {
    ARD_HIP_CHECK(ard::raise_lds_limit((const void*)kernel, (int)lds_bytes));
    raised = !dry_run();
  }
  ARD_LAUNCH_NAMED(launch_instance("gemm_direct_kernel", BM, BN, MODE), kernel, dim3((unsigned)grid_x), dim3(64 * NW), lds_bytes, stream, F);
  ARD_LAUNCH_CHECK("gemm_direct_kernel");
  return ARD_OK;
}
template <bool A_KC, bool B_KC, int BM, int BN, int NW, int MODE>
static int32_t launch_direct_kernel(const FastParams& F_in, int grid_x, hipStream_t stream) {
  FastParams F = F_in;
  if (F.splits < 1) F.splits = 1;
  const size_t lds_bytes = direct_lds_bytes(BM, BN, MODE);
  // class-free launches: the (split, tile) items are dealt to the XCDs inside the kernel
  if (F.tab.ncls == 0) grid_x = direct_plain_grid(F.total_tiles * (F.splits < 1 ? 1 : F.splits));
  // no lane may leave its operand: cheap envelope always, the exhaustive walk on request
  if (int32_t st = direct_envelope<A_KC, B_KC, BM, BN, MODE>(F)) return st;
  if constexpr (MODE != 3) {  // (MODE 3: the envelope is exact, whatever the list says)
    if (dry_run() || dev_knobs().prove_bounds) {
      DirectBounds b;
      if (int32_t st = direct_prove<A_KC, B_KC, BM, BN, NW, MODE>(F, grid_x, b)) return st;
      note_direct_bounds(b, F.a_elems * 2, F.b_elems * 2);
    }
  }
  constexpr int gk = direct_group_kind<A_KC, B_KC, BM, BN, NW, MODE>();
  if (gk >= 0 && batch_open() && batch_push_direct(gk, F, grid_x, lds_bytes)) return ARD_OK;
  return launch_direct_alone<A_KC, B_KC, BM, BN, NW, MODE>(F, grid_x, stream);
}

}  // namespace ard
