// Data gradient of a convolution whose output positions are partly dropped (row pattern of Section 5.2.1, block pattern of
// Section 5.2.2), bf16, filters that keep the image's size.
//
// dA[c, q] = sum over taps of Wt[., c, tap]^T dY[., q + pad - tap], and only kept positions of dY carry a gradient.  As a product
// over the positions of dA (the ordinary data gradient) a dropped position costs as much as a kept one: kept rows are
// scattered single positions under which no whole step of the contraction can be left out.  So the product runs over the
// kept positions of dY instead, tap by tap, and each tap's result is added where it belongs: a workgroup holds the sums of
// 16 channels of a few images (or a band of rows) in LDS, [position][16 channels], with a border that takes what falls
// outside, so that a tap is one constant distance.
//
// The copy of dY leaves its kept positions a second time, in the order the MFMAs take them (GradTiles): on the channels-last
// grid neighbouring lanes would read 16 bytes each of different positions (layer below, blocks of 112 positions: 108 instead
// of 79 us, the copy 27 instead of 41).  A wavefront takes up to 64 positions and keeps their channels in registers for
// all taps (128 registers at 256 channels); the weights of a tap (8 KB) pass through LDS, packed in MFMA order too
// (scatter_pack_body).
// Within a tap no two positions meet, between taps lies a barrier: the sums are added in the order of the taps and come
// out the same every time.  A tap's results are added under the MFMAs of the next, a lane taking four channels of a
// position: one 16-byte read and one write per tile (ds_add_f32 takes 192 clocks a wavefront whatever its addresses, a read
// and a write of 4 bytes 8, of 16 bytes 17).  Two workgroups share a CU, so that one loads its positions or stores its sums
// while the other multiplies.
#pragma once
#include "fast.hpp"

namespace ard {

constexpr int kSdLds = 80 * 1024, kSdMostLds = 160 * 1024;               // two workgroups per CU; one, for wide planes
constexpr int scatter_bufs(int ks) { return ks >= 6 ? 2 : 4; }           // taps of weights in LDS
constexpr int scatter_weight_bytes(int ks) { return scatter_bufs(ks) * ks * 1024; }
constexpr int kSdImages = 64, kSdTail = kSdImages * 8;                   // most images of a workgroup, their ranks

// Kept positions of dY in tiles of 16: [image][TI tiles][steps of 32 channels][64 lanes][8], lane l of a step holds channels
// 8 * (l >> 4) + e of position l & 15.  Position p of image n counts for column block cb if mask[(n * RB + p / x) * CB + cb]
// is not 0.  Bands of one position: the tiles of an image are made of its kept ones, in ascending order; cols: which they
// are, [image][16 * TI]; row_start: how many lie before every row, [image][H + 1].  Others (cols == NULL): tiles of
// neighbours, of which those that no column block keeps hold anything.
struct GradTiles {
  uint16_t* tiles;
  uint16_t* cols;
  int* row_start;
  const uint8_t* mask;
  int TI, RB, CB, x;
};
__device__ __forceinline__ bool grad_kept(const GradTiles& t, int n, int band, int cb) { return t.mask[((long)n * t.RB + band) * t.CB + cb] != 0; }

struct ScatterDataParams {
  const uint16_t* W;     // fragments [group of 16 channels][pass][tap][KS][64 lanes][8], see scatter_pack_body
  GradTiles t;           // dY
  uint16_t* dA;
  int N, C, H, W_, HW, steps;  // sizes of dA and dY, their plane, steps of 32 channels
  int kh, kw, ph, pw, taps, passes;  // passes of KS * 32 channels of dY
  int G, total, im, rows, bands;     // groups of 16 channels, workgroups, images or rows of dA per workgroup, bands of an image
  int Wl, tab_cap, lds_acc;          // slots of a row of sums, most tiles of a workgroup, bytes of the sums (and of where dead columns go)
  int width;                         // bytes per store of dA
  int lds_bytes;
  FastDiv by_groups, by_bands, by_hw, by_w, by_x, by_gpb;  // G, bands, HW, W_, x, groups per column block
};

// One wavefront's worth of packed weights per (group, pass, tap, step): lane l holds channel 16 * group + (l & 15) of dA and
// channels 32 * step + 8 * (l >> 4) + e of dY.
struct ScatterPackJob {
  const uint16_t* Wt;  // [Cout][C][taps]
  int C, Cout, taps, passes, ks, G;
  uint16_t* out;
  int blocks;  // workgroups of 256 threads: four fragments each (0: no job)
};

// Steps of a pass, passes and bytes of the packed weights: as few passes over the channels of dY as registers allow (256
// channels each), of equal depth.
__host__ __forceinline__ void scatter_passes(int C, int Cout, int taps, int& ks, int& passes, size_t& w_bytes) {
  const int g64 = (Cout + 63) / 64;
  passes = (g64 + 3) / 4;
  ks = 2 * ((g64 + passes - 1) / passes);
  w_bytes = (size_t)((C + 15) / 16) * passes * taps * ks * 1024;
}

// How the images are dealt to workgroups: as many whole images, or rows of one, as fit in LDS (every band reads 2 ph rows
// more than it writes: where that is more than half, one workgroup takes the whole LDS), but not so many that the chip's
// 512 places stay empty.  false: not even one row fits.
__host__ __forceinline__ bool scatter_units(ScatterDataParams& P, int ks, int lds = kSdLds) {
  const long room = lds - scatter_weight_bytes(ks) - kSdTail;
  auto slots = [&](long im, long nh) { return (im * (nh + P.kh - 1) * P.Wl + (P.kh - 1) * P.Wl + 2 * P.kw + 3) / 4 * 4; };
  auto fits = [&](long im, long rows) {
    const long nh = rows >= P.H ? P.H : (rows + 2 * P.ph < P.H ? rows + 2 * P.ph : P.H);
    return im <= kSdImages && im * (nh * P.W_ / 16 + 2) <= 256 && slots(im, nh) * 64 + (im * (nh * P.W_ / 16 + 2) + 1) * 4 <= room;
  };
  P.im = 1, P.rows = P.H;
  if (fits(1, P.H)) {
    while (P.im < P.N && fits(P.im + 1, P.H)) ++P.im;
    const long most = (long)P.N * P.G / 512;
    if (P.im > most) P.im = most < 1 ? 1 : (int)most;
  } else {
    while (P.rows > 0 && !fits(1, P.rows)) --P.rows;
    if (P.rows < 4 * P.ph && lds < kSdMostLds) return scatter_units(P, ks, kSdMostLds);
    if (P.rows < 1) return false;
  }
  if (P.im == 1 && (long)P.N * P.G < 512) {  // (a band of less than two filters costs more than it brings)
    const int want = (int)((512 + (long)P.N * P.G - 1) / ((long)P.N * P.G)), rows = (P.H + want - 1) / want;
    const int least = 2 * P.kh < P.H ? 2 * P.kh : P.H;
    if (rows < P.rows) P.rows = rows > least ? rows : (least < P.rows ? least : P.rows);
  }
  if (P.rows < P.H) {
    P.rows = (P.H + (P.H + P.rows - 1) / P.rows - 1) / ((P.H + P.rows - 1) / P.rows);  // (bands of equal height)
    for (int m = 8; m > 1; m /= 2)  // (that start on pieces of 16 bytes, or 8 or 4, if the planes do)
      if (P.HW % m == 0) {
        int r = P.rows;
        while (r > 1 && r * P.W_ % m) --r;
        if (r * P.W_ % m == 0 && r * 8 >= P.rows * 7) { P.rows = r; break; }
      }
  }
  P.bands = (P.H + P.rows - 1) / P.rows;
  const int nh = P.rows >= P.H ? P.H : (P.rows + 2 * P.ph < P.H ? P.rows + 2 * P.ph : P.H);
  P.lds_acc = (int)slots(P.im, nh) * 64;
  P.tab_cap = (P.im * (nh * P.W_ / 16 + 2) + 1) / 2 * 2;
  P.lds_bytes = scatter_weight_bytes(ks) + P.lds_acc + P.tab_cap * 4 + kSdTail;
  return true;
}
__device__ __forceinline__ void scatter_pack_body(const ScatterPackJob& j, int block) {
  const int f = block * 4 + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int per_group = j.passes * j.taps * j.ks, g = f / per_group;
  if (g >= j.G) return;
  int r = f - g * per_group;
  const int pass = r / (j.taps * j.ks);
  r -= pass * j.taps * j.ks;
  const int tap = r / j.ks, step = r - tap * j.ks;
  const int c = g * 16 + (lane & 15), co = (pass * j.ks + step) * 32 + (lane >> 4) * 8;
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (c < j.C && co + e < j.Cout) w[e >> 1] |= (uint32_t)j.Wt[((long)(co + e) * j.C + c) * j.taps + tap] << ((e & 1) * 16);
  reinterpret_cast<uint4*>(j.out)[(long)f * 64 + lane] = make_uint4(w[0], w[1], w[2], w[3]);
}

template <int N> __device__ __forceinline__ void wait_lgkm() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N > 15 ? 15 : N) : "memory"); }

// Byte of 4 channels of a slot.  Neighbouring slots hold them in different order, and change places in fours: the same
// channels of four neighbours, and all channels of four slots eight apart (the way out), lie in different banks.
__device__ __forceinline__ unsigned scatter_at(unsigned slot, unsigned kg) { return (slot ^ (slot >> 3 & 3u)) * 64u + ((kg ^ slot) & 3u) * 16u; }
// (Reads and writes of the sums as asm: the compiler, which takes any LDS-direct load in flight for one to the same
// address, would wait for all of them first.)
__device__ __forceinline__ void scatter_write(unsigned byte_addr, f32x4_t v) { asm volatile("ds_write_b128 %0, %1" ::"v"(byte_addr), "v"(v) : "memory"); }

// KS: 32-deep steps of a pass (2, 4, 6 or 8).
template <int KS>
__global__ __launch_bounds__(256, 2) void conv_scatter_data_kernel(const ScatterDataParams P) {
  extern __shared__ uint4 sd_lds[];
  constexpr int NBUF = scatter_bufs(KS), LPT = (KS + 3) / 4, WB = KS * 64;  // loads of a wavefront per tap, 16-byte pieces of a tap
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  touch_args<(int)(sizeof(ScatterDataParams) / 64)>(P);
  // XCD x takes the x-th eighth of the units; the groups of a unit follow each other and share its positions in L2
  const int xcd = (int)blockIdx.x & 7, lo = (int)((long)xcd * P.total / 8), hi = (int)((long)(xcd + 1) * P.total / 8);
  const int L = lo + ((int)blockIdx.x >> 3);
  if (L >= hi) return;
  const int u = (int)fdiv((uint32_t)L, P.by_groups), g = L - u * P.G;
  const int ui = (int)fdiv((uint32_t)u, P.by_bands), band = u - ui * P.bands;
  const int n0 = ui * P.im, imgs = imin(P.im, P.N - n0);
  const int r0 = band * P.rows, r1 = imin(r0 + P.rows, P.H);         // rows of dA
  const int h0 = imax(r0 - P.ph, 0), h1 = imin(r1 + P.ph, P.H);      // rows of dY that reach them
  const int slots_img = (h1 - h0 + P.kh - 1) * P.Wl;
  char* const acc = reinterpret_cast<char*>(sd_lds) + NBUF * WB * 16;
  uint32_t* const tab = reinterpret_cast<uint32_t*>(acc + P.lds_acc);  // tiles of the unit: image of the unit << 16 | tile of the image
  int2* const ranks = reinterpret_cast<int2*>(tab + P.tab_cap);  // first kept position of an image's rows, and the first behind them
  int* const counts = reinterpret_cast<int*>(ranks);
  // weights: tap tile i of the stream (pass by pass, for every chunk of positions anew)
  const int tiles = P.passes * P.taps;
  const char* const Wg = reinterpret_cast<const char*>(P.W) + (long)g * tiles * (WB * 16) + lane * 16;
  int next = 0, ahead = 0;  // tile of the next loads, its buffer
  auto load_weights = [&]() {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int f = (wave + 4 * i) % KS;  // (a remainder is loaded twice)
      __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(Wg + (next * KS + f) * 1024), ARD_LDS_PTR(sd_lds + ahead * WB + f * 64), 16, 0, 0);
    }
    next = next + 1 < tiles ? next + 1 : 0;
    ahead = (ahead + 1) % NBUF;
  };
#pragma unroll
  for (int i = 0; i < NBUF; ++i) load_weights();
  // the tiles that hold a kept position of the unit's rows
  const int cb = (int)fdiv((uint32_t)g, P.by_gpb), pa = h0 * P.W_, pb = h1 * P.W_;
  const auto zero_sums = [&]() {
    for (int i = tid; i < P.lds_acc / 16; i += 256) reinterpret_cast<uint4*>(acc)[i] = make_uint4(0, 0, 0, 0);
  };
  int ntiles = 0;
  if (P.t.cols) {
    // (every wavefront for itself: a lane per image)
    const int* const rs = P.t.row_start + (long)(n0 + imin(lane, imgs - 1)) * (P.H + 1);
    const int k0 = rs[h0], k1 = rs[h1];
    zero_sums();
    const int t0 = k0 >> 4, n = lane < imgs && k1 > k0 ? ((k1 + 15) >> 4) - t0 : 0;
    int incl = n;
    for (int o = 1; o < imgs; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      incl += lane >= o ? v : 0;
    }
    ntiles = __builtin_amdgcn_readlane(incl, imgs - 1);
    if (wave == 0 && lane < imgs) {
      ranks[lane] = make_int2(k0, k1);
      for (int i = 0; i < n; ++i) tab[incl - n + i] = (uint32_t)(lane << 16 | (t0 + i));
    }
  } else {
    // (a thread per tile)
    const int ta = pa >> 4, per = ((pb + 15) >> 4) - ta, im = P.im > 1 ? tid / per : tid >= per, t = ta + tid - im * per;
    bool k = false;
    if (im < imgs) {
      const int p0 = imax(t * 16, pa), p1 = imin(t * 16 + 16, pb) - 1;
      for (int b = (int)fdiv((uint32_t)p0, P.by_x); b <= (int)fdiv((uint32_t)p1, P.by_x); ++b) k |= grad_kept(P.t, n0 + im, b, cb);
    }
    zero_sums();
    const unsigned long long has = __ballot(k);
    if (lane == 0) counts[wave] = __builtin_popcountll(has);
    __syncthreads();
    int at = __builtin_popcountll(has & ((1ull << lane) - 1));
    for (int w = 0; w < 4; ++w) {
      at += w < wave ? counts[w] : 0;
      ntiles += counts[w];
    }
    if (k) tab[at] = (uint32_t)(im << 16 | t);
  }
  ntiles = __builtin_amdgcn_readfirstlane(ntiles);
  __syncthreads();  // (waits for the weights of the first taps as well)
  const int chunks = (ntiles + 15) >> 4, total = chunks * tiles;
  int j = 0, buf = 0;  // tap of the stream, its buffer
  const int col = lane & 15, kg = lane >> 4;
  const unsigned wbase = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)sd_lds) + (unsigned)lane * 16u;
  const unsigned abase = wbase - (unsigned)lane * 16u + (unsigned)(NBUF * WB * 16);
  const char* const dy = reinterpret_cast<const char*>(P.t.tiles) + (long)n0 * P.t.TI * P.steps * 1024;
  const int steps = P.steps;
  const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
  Frag fb[2];
  auto chunk = [&](auto ntc, int c) {
    // sums are read in the first GR steps, PER tiles at a time, and written a step later
    constexpr int NT = decltype(ntc)::value, PER = KS > 3 ? (NT + KS - 4) / (KS - 3) : NT;
    // Column n of a tile is a position, rows are channels: a lane has four channels of one position.
    uint32_t e[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) e[i] = tab[imin(c * 16 + i * 4 + wave, ntiles - 1)];
    unsigned from[NT], to[NT];
    int p[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      e[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)e[i]);
      const unsigned tile = (e[i] >> 16) * (unsigned)P.t.TI + (e[i] & 0xffffu);
      from[i] = tile * (unsigned)steps * 1024u + (unsigned)lane * 16u;
      p[i] = P.t.cols ? P.t.cols[(long)n0 * P.t.TI * 16 + tile * 16u + (unsigned)col] : (int)(e[i] & 0xffffu) * 16 + col;
    }
    bf16x8_t a[NT][KS];
    auto load_positions = [&](int pass) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          uint4 v = make_uint4(0, 0, 0, 0);
          if (pass * KS + s < steps) v = *reinterpret_cast<const uint4*>(dy + (from[i] + (unsigned)((pass * KS + s) * 1024)));
          a[i][s] = __builtin_bit_cast(bf16x8_t, v);
        }
    };
    load_positions(0);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int im = (int)(e[i] >> 16);
      bool kept = c * 16 + i * 4 + wave < ntiles;
      if (P.t.cols) {
        const int2 r = ranks[im];
        const int rank = (int)(e[i] & 0xffffu) * 16 + col;
        kept = kept & (rank >= r.x) & (rank < r.y);
      } else {
        const int q = imin(imax(p[i], pa), pb - 1);
        kept = kept & (p[i] == q) & grad_kept(P.t, n0 + im, (int)fdiv((uint32_t)q, P.by_x), cb);
      }
      const int h = (int)fdiv((uint32_t)p[i], P.by_w), w = p[i] - h * P.W_;
      to[i] = (unsigned)(kept ? im * slots_img + (h - h0) * P.Wl + w : imgs * slots_img + P.kw);  // (columns that are no position: a place of their own)
    }
    for (int pass = 0; pass < P.passes; ++pass) {
      if (pass) load_positions(pass);
      f32x4_t even[NT], odd[NT];
      auto read = [&](auto sc, int b) {
        constexpr int S = decltype(sc)::value;
        lds_read_b128<S * 1024>(fb[S & 1].v, wbase + (unsigned)(b * WB * 16));
      };
      Frag held[NT];
      unsigned at[NT];
      auto fetch = [&](int i, unsigned off) {
        at[i] = abase + scatter_at(to[i] + off, (unsigned)kg);
        lds_read_b128<0>(held[i].v, at[i]);
      };
      auto put = [&](f32x4_t (&sum)[NT], int i) {
        frag_wait<true>(held[i]);
        f32x4_t v = __builtin_bit_cast(f32x4_t, held[i].v);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += sum[i][e];
        scatter_write(at[i], v);
      };
      // one tap; `prev`: the sums of the tap before, to be added at `off`
      auto tap = [&](auto firstc, bool last, f32x4_t (&sum)[NT], f32x4_t (&prev)[NT], unsigned off) {
        constexpr bool FIRST = decltype(firstc)::value;
        const int nb = (buf + 1) % NBUF;
        static_for<KS>([&](auto sc) {
          constexpr int S = decltype(sc)::value;
          if constexpr (!FIRST && KS == 2 && S == 0) {
#pragma unroll
            for (int i = 0; i < NT; ++i) fetch(i, off);
          }
          wait_lgkm<KS == 2 && S == 0 && !FIRST ? 0 : 1>();  // (all but the youngest read of weights)
          frag_wait<true>(fb[S & 1]);
#pragma unroll
          for (int i = 0; i < NT; ++i)
            sum[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_value<true>(fb[S & 1]), a[i][S], S == 0 ? zero : sum[i], 0, 0, 0);
          if constexpr (!FIRST) {
#pragma unroll
            for (int i = KS == 2 ? 0 : (S > 0 ? (S - 1) * PER : 0); i < NT && i < (KS == 2 ? NT - S * NT : S * PER); ++i) put(prev, i);
            if constexpr (KS > 2) {
#pragma unroll
              for (int i = S * PER; i < NT && i < (S + 1) * PER; ++i) fetch(i, off);
            }
          }
          if constexpr (S == KS - 2) {
            // this wavefront's reads of the tap and its additions are done, its share of the next tap's weights is there
            wait_lgkm<0>();
            if (j + NBUF - 1 < total) wait_vmcnt<(NBUF - 2) * LPT>();
            else wait_vmcnt<0>();
            wg_barrier();
            if (j + NBUF < total) load_weights();
          }
          if constexpr (S + 2 < KS) read(std::integral_constant<int, (S + 2) % KS>{}, buf);
          else if (!last) read(std::integral_constant<int, (S + 2) % KS>{}, nb);
        });
        ++j, buf = nb;
      };
      read(std::integral_constant<int, 0>{}, buf);
      read(std::integral_constant<int, 1>{}, buf);
      unsigned off = 0;
      int s = 0;  // of the tap whose sums are pending; its filter column
      auto advance = [&]() {
        ++s;
        ++off;
        if (s == P.kw) s = 0, off += (unsigned)(P.Wl - P.kw);
      };
      const int taps = P.taps;
      tap(std::true_type{}, taps == 1, even, even, 0u);
      int t = 1;
      for (; t + 1 < taps; t += 2) {
        tap(std::false_type{}, false, odd, even, off);
        advance();
        tap(std::false_type{}, t + 2 == taps, even, odd, off);
        advance();
      }
      auto flush = [&](f32x4_t (&sum)[NT]) {
#pragma unroll
        for (int i = 0; i < NT; ++i) fetch(i, off);
        wait_lgkm<0>();
#pragma unroll
        for (int i = 0; i < NT; ++i) put(sum, i);
      };
      if (t < taps) {
        tap(std::false_type{}, true, odd, even, off);
        advance();
        flush(odd);
      } else {
        flush(even);
      }
    }
  };
  for (int c = 0; c < chunks; ++c) {
    const int n = imin(ntiles - c * 16, 16);
    if (n > 12) chunk(std::integral_constant<int, 4>{}, c);
    else if (n > 8) chunk(std::integral_constant<int, 3>{}, c);
    else if (n > 4) chunk(std::integral_constant<int, 2>{}, c);
    else chunk(std::integral_constant<int, 1>{}, c);
  }
  wait_lgkm<0>();
  __syncthreads();
  // a thread takes four channels and E neighbouring positions
  const int rows = r1 - r0, out_per = rows * P.W_, out_n = imgs * out_per, kq = tid & 3, ch = g * 16 + kq * 4;
  auto store = [&](auto unit) {
    using U = decltype(unit);
    constexpr int E = (int)sizeof(U) / 2;
    for (int q = (tid >> 2) * E; q < out_n; q += 64 * E) {
      const int im = P.im > 1 ? (int)fdiv((uint32_t)q, P.by_hw) : 0, rem = q - im * out_per;
      int h = (int)fdiv((uint32_t)rem, P.by_w), w = rem - h * P.W_;
      unsigned slot = (unsigned)(im * slots_img + (r0 + P.ph - h0 + h) * P.Wl + P.pw + w);
      float4 f[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        f[e] = *reinterpret_cast<const float4*>(acc + scatter_at(slot, (unsigned)kq));
        ++slot;
        if (++w == P.W_) w = 0, slot += (unsigned)(P.Wl - P.W_);
      }
      uint16_t* const dst = P.dA + ((long)(n0 + im) * P.C + ch) * P.HW + r0 * P.W_ + rem;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (ch + k >= P.C) break;
        auto v = [&](int e) { return k == 0 ? f[e].x : k == 1 ? f[e].y : k == 2 ? f[e].z : f[e].w; };
        if constexpr (E == 1) {
          dst[(long)k * P.HW] = f32_to_bf16_bits(v(0));
        } else {
          struct { uint32_t w[E / 2]; } words;
#pragma unroll
          for (int e = 0; e < E / 2; ++e) words.w[e] = pack_bf16x2(v(2 * e), v(2 * e + 1));
          *reinterpret_cast<U*>(dst + (long)k * P.HW) = __builtin_bit_cast(U, words);
        }
      }
    }
  };
  if (P.width == 16) store(uint4{});
  else if (P.width == 8) store(uint2{});
  else if (P.width == 4) store(uint32_t{});
  else store(uint16_t{});
}

// (conv_kept.hip)
int32_t launch_conv_scatter(int ks, const ScatterDataParams& P, hipStream_t stream);

}  // namespace ard
