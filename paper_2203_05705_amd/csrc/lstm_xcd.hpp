// Recurrences of the LSTM with a batch block per XCD (included by lstm.hip, after the helpers of the other one-launch forms).
#pragma once

namespace ard {

// What bounds a recurrence is the exchange from one step to the next.  RB batch rows are one block (8 while eight such
// blocks hold the batch, else 16), and all workgroups of a block run on one XCD (the dispatcher deals workgroups
// round-robin, block bb takes XCD bb): what they exchange in a step, h_t forward and dG_t backward, never leaves that XCD's
// L2.  From a store to the load that sees it 370 ns pass there, 510 if the store is written through to memory, 650 to
// another XCD.
//
// A workgroup owns UW kept units (16 up to 512 kept units, 24 up to 768: 32 workgroups at most, one per CU) and has
// wavefronts that multiply and four that run the cell; the recurrent weights stay in registers.  The rows arrive at the
// product wavefronts in the order their MFMAs take them (what a cell wavefront stores is a whole 128-byte line of that
// image), each leaves its partial tile in LDS, one barrier, the cell wavefronts add the partial tiles, run the cell, store
// what the others wait for, and then everything else.  A product wavefront stores nothing, so its loads wait for nobody's
// stores (vmcnt counts both in order).
//
// Where the workgroups of a block really run is read from the hardware at the start (lx_meet): on one XCD results are
// stored into its L2; if they are spread, device-scope stores make the same loads correct at the old price.
//
// No workgroup waits for one that may not have a CU: two recurrences on two streams may share an XCD's CUs so that neither
// ever has all of its own.  A workgroup's part of a block is a seat; when some are still free after kLxPatience polls, those
// that are there take them as well, and do their parts of a step one after the other with weights from memory.  One that
// comes too late leaves.  (750 units, B = 20, 35 steps, with 31, 16 and 1 of 32 workgroups: forward 84 -> 257, 579 and
// 4800 us, backward 146 -> 557, 1170 and 10200.)
//
// Recurrences with staging wavefronts -> these, us: 512 kept units, B = 128, 64 steps: forward 204 -> 114, backward
// 237 -> 158; 750 units, B = 20, 35 steps: 113 -> 67 and 136 -> 88 (with 16 rows per block 95 and 142: half of every
// operand and of the cells would be padding).  Eight product wavefronts instead of four at 512 units forward, or a higher
// priority of the cell wavefronts: nothing.
constexpr int kLxBlocks = 8, kLxSeats = 32;  // most batch blocks, most workgroups of one
constexpr int kLxBwdWaves = 8;               // wavefronts that multiply, backward and forward
constexpr int lx_fwd_waves(int uw) { return uw == 16 ? 4 : 8; }

// Byte of (row, unit) in the [RB rows x UW units] image of one workgroup, bf16: groups of 8 units are 16-byte pieces (a
// lane's MFMA operand); 4 rows x 16 units are one line (a wavefront's cells), the last 8 units of 24 follow in lines of
// 8 rows.  (The two groups of units change places from row 8 on: the 16 rows an LDS read takes at a time then lie in
// different banks.)
template <int RB> __device__ __forceinline__ int lx_at(int row, int unit) {
  return unit < 16 ? (row >> 2) * 128 + (((unit >> 3) ^ (row >> 3)) & 1) * 64 + (row & 3) * 16 + (unit & 7) * 2 : RB * 32 + row * 16 + (unit & 7) * 2;
}
// cell `c` of a workgroup's RB * UW cells, in the order of the image
template <int RB> __device__ __forceinline__ void lx_cell(int c, int& row, int& unit) {
  const int d = c - RB * 16;
  row = d < 0 ? c >> 4 : d >> 3;
  unit = d < 0 ? c & 15 : 16 + (d & 7);
}
// 1 / d for d >= 1: the hardware's reciprocal and one Newton step (which makes a NaN of an infinity's 0)
__device__ __forceinline__ float lx_rcp(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return d < 3.0e38f ? fmaf(fmaf(-d, r, 1.0f), r, r) : (d != d ? d : r);
}
__device__ __forceinline__ float lx_sigmoid(float z) { return lx_rcp(1.0f + __expf(-z)); }
// tanh without branches: a polynomial fitted to (tanh(x) / x - 1) / x^2 on [0, 1.1] (2e-9), 1 - 2 / (1 + e^2x) beyond.
// Against 64 bits over 4 M values up to 20: at most 1.11 ulp, 0.215 in the mean (tanhf 1.34 and 0.216, and a training step of
// 64 time steps of 1024 units at batch 128 531 instead of 526 us).
__device__ __forceinline__ float lx_tanh(float x) {
  const float y = fabsf(x), s = x * x;
  float p = 9.130840044e-05f;
  p = fmaf(s, p, -0.0007175668143f);
  p = fmaf(s, p, 0.00287373201f);
  p = fmaf(s, p, -0.008419346064f);
  p = fmaf(s, p, 0.02170202322f);
  p = fmaf(s, p, -0.05393234268f);
  p = fmaf(s, p, 0.1333295405f);
  p = fmaf(s, p, -0.3333331943f);
  const float low = fmaf(x * s, p, x), high = copysignf(fmaf(-2.0f, lx_rcp(1.0f + __expf(2.0f * y)), 1.0f), x);
  return y < 1.1f ? low : high;
}
// The workgroups of a block take their seats, tell each other which XCD they run on, and take the seats of those that are
// not there.  Returns the number of seats taken, -1 when forced to give up; `local`: all of them are on one XCD.
constexpr int kLxPatience = 256;  // polls of half a microsecond or more: about what a recurrence takes
__device__ __forceinline__ int lx_meet(int* seat, int S, int s, int lane, long limit, int* err, int* taken, int& local) {
  unsigned x;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
  const int mine = (int)(x & 0xffu) + 1;
  auto take = [&](int k) {
    int was = 0;
    if (lane == 0) __hip_atomic_compare_exchange_strong(seat + k, &was, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_amdgcn_readfirstlane(was) == 0;
  };
  if (limit < 0) {  // (the host's way to force the give-up path)
    __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return -1;
  }
  if (!take(s)) return 0;
  if (lane == 0) taken[0] = s;
  for (int n = 1, polls = 0;; ++polls) {
    const int v = lane < S ? __hip_atomic_load(seat + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : mine;
    const uint64_t free = __ballot(v == 0);
    local = __all(v == mine);
    if (!free) return n;
    if (polls < kLxPatience) continue;
    // each its own share of the free ones: in the order of those that are there, and not the next one at once
    const int rank = __builtin_popcountll(__ballot(lane < s && v != 0)) % __builtin_popcountll(free);
    const bool wanted = (free >> lane & 1) && __builtin_popcountll(free & ((1ull << lane) - 1)) == rank;
    const int k = __builtin_ctzll(__ballot(wanted));
    polls -= 8;
    if (!take(k)) continue;
    if (lane == 0) taken[n] = k;
    ++n;
  }
}
// a result and its neighbour's (lane ^ 1) as the word that the even one stores; every NaN becomes 0x7fc0 (kUnwritten)
__device__ __forceinline__ unsigned lx_word(float x) {
  if (x != x) x = __uint_as_float(0x7fc00000u);
  const float y = __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0xB1, 0xF, 0xF, true));
  return pack_bf16x2(x, y);
}
__device__ __forceinline__ void lx_store(char* base, unsigned at, unsigned v, bool local) {
  unsigned* const p = reinterpret_cast<unsigned*>(base + at);
  if (local) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// This lane's number, found anew: what a workgroup with several seats derives from it in a loop is worked out there, where
// the usual loop needs the registers.
__device__ __forceinline__ int lx_lane() {
  int zero = 0;
  asm volatile("" : "+v"(zero));
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (unsigned)zero));
}
// Waits for what such a loop has loaded, known to the compiler: where its path joins the usual one, which counts the loads
// and stores that may stay in flight, none of it is left (else each step waited for all of its stores: 10 us a pass).
__device__ __forceinline__ void lx_landed() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)
__device__ __forceinline__ unsigned lx_min(unsigned a, unsigned b) { return a < b ? a : b; }
__device__ __forceinline__ unsigned lx_max3(unsigned a, unsigned b, unsigned c) {
  const unsigned m = a > b ? a : b;
  return m > c ? m : c;
}
// Loads N pieces per lane until nothing in them is unwritten (kUnwritten is the largest word).  False: gave up.
template <int N>
__device__ __forceinline__ bool lx_wait(__amdgpu_buffer_rsrc_t buf, const unsigned (&at)[N], lp_u32x4 (&v)[N], long limit, int* err) {
  long spins = 0;
  for (;;) {
    unsigned most = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = lp_load(buf, at[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) most = lx_max3(lx_max3(most, v[i].x, v[i].y), v[i].z, v[i].w);
    if (!__any(most == kUnwritten)) return true;
    if (lp_give_up(spins, limit, err)) return false;
  }
}

// KW: 32-wide slices of the contraction per product wavefront.
template <int RB, int UW, int KW>
__global__ __launch_bounds__(64 * (lx_fwd_waves(UW) + 4)) void lstm_xcd_fwd_kernel(const LstmPersist P) {
  constexpr int NM = lx_fwd_waves(UW), BLK = RB * UW * 2, NT = UW / 4, NP = (RB * UW + 255) / 256, RED = RB * UW;
  extern __shared__ uint4 lp_lds[];
  __shared__ int go_s[2], local_s, seats_s, seat_s[kLxSeats];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bb = (int)blockIdx.x & 7, s = (int)blockIdx.x >> 3, nbb = (P.B + RB - 1) / RB, S = P.S;
  if (bb >= nbb || (P.seats && s >= P.seats)) return;
  const int Hp = P.Hp, B = P.B, H = P.H;
  float4* const red = reinterpret_cast<float4*>(lp_lds);             // [2][NM][RED] sums of the four gates of a cell
  char* const ex = reinterpret_cast<char*>(P.hc) + (long)bb * S * BLK;  // this block's images of step 0
  const long ex_step = (long)nbb * S * BLK;
  if (tid == 0) go_s[0] = go_s[1] = 1;
  if (wave == NM) {
    int local = 0;
    const int m = lx_meet(P.counters + bb * kLxSeats, S, s, lane, P.spin_limit, P.err, seat_s, local);
    if (lane == 0) seats_s = m, local_s = local;
  }
  if (wave < NM) {
    const int n = lane & 15, kg = lane >> 4;
    // gate columns of this workgroup: tiles 0 .. 3 the gates of its first 16 units; 4 and 5 (24 units) gates 0 | 1 and
    // 2 | 3 of its last 8
    bf16x8_t wf[KW][NT];
    auto weights = [&](int seat, int n, int kg) {
#pragma unroll
      for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
          const int k = ((wave * KW + i) * 4 + kg) * 8;
          const int gate = tt < 4 ? tt : 2 * (tt - 4) + (n >> 3), unit = seat * UW + (tt < 4 ? n : 16 + (n & 7));
          uint4 v = make_uint4(0, 0, 0, 0);
          if (k < Hp && unit < Hp) v = *reinterpret_cast<const uint4*>(P.Wh + ((long)gate * Hp + unit) * Hp + k);
          wf[i][tt] = __builtin_bit_cast(bf16x8_t, v);
        }
    };
    weights(s, n, kg);
    unsigned at[KW];
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      const int g8 = (wave * KW + i) * 4 + kg, ws = g8 / (UW / 8);  // group of 8 units, its writer (none: zero weights)
      at[i] = (unsigned)((ws < S ? ws * BLK : 0) + lx_at<RB>(n & (RB - 1), (g8 - ws * (UW / 8)) * 8));
    }
    // (`it` counts the steps of all seats: what go_s and red hold of one stays until the next but one)
    const char* src = ex;  // images of the step before
    auto product = [&](int t, int it) {
      if (t > 0) {
        lp_u32x4 v[KW];
        if (!lx_wait<KW>(lp_buffer(src, (unsigned)(S * BLK)), at, v, P.spin_limit, P.err)) go_s[it & 1] = 0;
        f32x4_t acc[NT];
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[tt][e] = 0.0f;
#pragma unroll
        for (int i = 0; i < KW; ++i)
#pragma unroll
          for (int tt = 0; tt < NT; ++tt) acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, v[i]), wf[i][tt], acc[tt], 0, 0, 0);
        // lane holds column n, rows 4 kg + e; the gates of a cell side by side (24 units, the last 8: gates 0 2 | 1 3)
        float4* const mine = red + ((it & 1) * NM + wave) * RED;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = 4 * kg + e;
          if (RB < 16 && row >= RB) continue;  // (rows beyond the block repeat its rows)
          mine[row * 16 + n] = make_float4(acc[0][e], acc[1][e], acc[2][e], acc[3][e]);
          if constexpr (UW == 24)
            reinterpret_cast<float2*>(mine + RB * 16 + row * 8 + (n & 7))[n >> 3] = make_float2(acc[4][e], acc[5][e]);
        }
      }
      lp_barrier();
      return __builtin_amdgcn_readfirstlane(go_s[it & 1]) != 0;  // uniform: every wavefront reads it behind the same barrier
    };
    lp_barrier();
    const int seats = __builtin_amdgcn_readfirstlane(seats_s);  // (0 and -1: nothing to do)
    for (int it = 0, t = 0, i = 0; t < P.T && seats > 0; ++it) {
      if (!product(t, it)) return;
      if (++i == seats) i = 0, src += t > 0 ? ex_step : 0, ++t;
      if (seats > 1) {
        const int l = lx_lane();
        weights(__builtin_amdgcn_readfirstlane(seat_s[i]), l & 15, l >> 4);
        lx_landed();
      }
    }
    return;
  }
  const int c0 = tid - 64 * NM;
  int row[NP], j[NP], u[NP], z_lo[NP], z_hi[NP];
  unsigned at[NP], zx_at[NP];  // byte of the cell's word in the image, its place in a row block of Gx
  uint32_t mask[NP];           // all ones of a kept cell
  bool kept[NP], live[NP], last8[NP];
  float c_reg[NP], zx[NP][4];
  auto cells = [&](int seat, int c0) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int c = p * 256 + c0;
      int ul;
      lx_cell<RB>(c, row[p], ul);
      live[p] = c < RB * UW;
      last8[p] = ul >= 16;
      j[p] = seat * UW + ul;  // compact unit
      at[p] = (unsigned)lx_at<RB>(row[p], ul) & ~3u;
      kept[p] = live[p] && j[p] < P.Hk;
      mask[p] = kept[p] ? ~0u : 0u;
      asm("" : "+v"(mask[p]));  // (or a branch comes of it)
      zx_at[p] = (unsigned)(imin(bb * RB + imin(row[p], RB - 1), B - 1) * 4 * Hp + imin(j[p], Hp - 1));  // (clamped: never used)
      u[p] = P.off + j[p] * P.step;  // physical unit
      // zeros of the dropped units this thread owns: the rest of its group [j*step, (j+1)*step), the last kept unit also
      // the tail up to H
      z_lo[p] = j[p] * P.step, z_hi[p] = !kept[p] ? z_lo[p] : (j[p] == P.Hk - 1 ? H : z_lo[p] + P.step);
      c_reg[p] = 0.0f;
    }
  };
  auto fetch_zx = [&](int t) {
    const float* Gt = P.Gx + (long)t * B * 4 * Hp;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int g = 0; g < 4; ++g) zx[p][g] = Gt[zx_at[p] + (unsigned)(g * Hp)];
  };
  bool local;
  char* img = ex;  // images of the step
  auto cell = [&](int t, int it, int seat, bool ahead) {
    char* const out = img + seat * BLK;
    // (here: the compiler would wait for these loads, and for the stores behind them, behind the barrier)
#pragma unroll
    for (int p = 0; p < NP; ++p) asm volatile("" : "+v"(zx[p][0]), "+v"(zx[p][1]), "+v"(zx[p][2]), "+v"(zx[p][3]));
    lp_barrier();
    if (!__builtin_amdgcn_readfirstlane(go_s[it & 1])) return false;
    float gi[NP], gf[NP], gg[NP], go[NP], hv[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (!live[p]) continue;
      float z[4] = {zx[p][0], zx[p][1], zx[p][2], zx[p][3]};
      if (t > 0) {
        const float4* src = red + (it & 1) * NM * RED + p * 256 + c0;
        float4 a[NM];
#pragma unroll
        for (int w = 0; w < NM; ++w) a[w] = src[w * RED];
#pragma unroll
        for (int w = NM / 2; w > 0; w >>= 1)
#pragma unroll
          for (int i = 0; i < w; ++i) a[i].x += a[i + w].x, a[i].y += a[i + w].y, a[i].z += a[i + w].z, a[i].w += a[i + w].w;
        z[0] += a[0].x, z[1] += last8[p] ? a[0].z : a[0].y, z[2] += last8[p] ? a[0].y : a[0].z, z[3] += a[0].w;
      }
      gi[p] = lx_sigmoid(z[0]), gf[p] = lx_sigmoid(z[1]), gg[p] = lx_tanh(z[2]), go[p] = lx_sigmoid(z[3]);
      const float cv = gf[p] * c_reg[p] + gi[p] * gg[p];
      c_reg[p] = cv;
      hv[p] = go[p] * lx_tanh(cv);
      // (the padding units store their zero; rows beyond the batch are stored like any other: the image is waited for as
      // a whole)
      const unsigned word = lx_word(__uint_as_float(__float_as_uint(hv[p]) & mask[p]));
      if (!(c0 & 1)) lx_store(out, at[p], word, local);
    }
    if (ahead && t + 1 < P.T) fetch_zx(t + 1);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int r = bb * RB + row[p];
      if (!kept[p] || r >= B) continue;
      float* ga = P.gates + ((long)t * B + r) * 4 * H;
      float* const pc = P.c + ((long)t * B + r) * H;
      uint16_t* const ph = P.h + ((long)t * B + r) * H;
      ga[u[p]] = gi[p], ga[H + u[p]] = gf[p], ga[2 * H + u[p]] = gg[p], ga[3 * H + u[p]] = go[p];
      pc[u[p]] = c_reg[p];
      ph[u[p]] = f32_to_bf16_bits(hv[p]);
      for (int uz = z_lo[p]; uz < z_hi[p]; ++uz) {
        if (uz == u[p]) continue;
        ga[uz] = ga[H + uz] = ga[2 * H + uz] = ga[3 * H + uz] = 0.0f;
        pc[uz] = 0.0f;
        ph[uz] = 0;
      }
    }
    return true;
  };
  cells(s, c0);
  fetch_zx(0);
  lp_barrier();
  local = local_s != 0 && !P.spread;
  const int seats = __builtin_amdgcn_readfirstlane(seats_s);
  for (int it = 0, t = 0, i = 0, seat = s; t < P.T && seats > 0; ++it) {
    if (!cell(t, it, seat, seats == 1)) return;
    if (++i == seats) i = 0, ++t, img += ex_step;
    if (seats > 1 && t < P.T) {
      seat = __builtin_amdgcn_readfirstlane(seat_s[i]);
      cells(seat, (wave - NM) * 64 + lx_lane());
      fetch_zx(t);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        if (t > 0 && kept[p] && bb * RB + row[p] < B) c_reg[p] = P.c[((long)(t - 1) * B + bb * RB + row[p]) * H + u[p]];
      lx_landed();
    }
  }
}

// KW as above.  The rows of a step, all 4 Hp gate columns of them, come through LDS: 64 KB a workgroup at 512 kept units, which eight
// wavefronts fetch in 770 clocks past the registers, in 1120 through them, and four in 1720.
template <int RB, int UW, int KW>
__global__ __launch_bounds__(64 * (kLxBwdWaves + 4)) void lstm_xcd_bwd_kernel(const LstmPersistBwd P) {
  constexpr int NM = kLxBwdWaves, GB = RB * UW * 2, BLK = 4 * GB, NB = UW / 16 + (UW % 16 > 0), NP = (RB * UW + 255) / 256, PITCH = UW + 4;
  constexpr int SHARE = KW * RB * 64, NL = SHARE / 1024, NOFF = UW == 16 ? 1 : 3;  // bytes of a wavefront's share, its loads
  constexpr int NA = UW == 16 ? 4 : 2;
  static_assert(SHARE % 1024 == 0 && SHARE % BLK == 0, "whole loads, whole writers");
  extern __shared__ uint4 lp_lds[];
  __shared__ int go_s[2], local_s, seats_s, seat_s[kLxSeats];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bb = (int)blockIdx.x & 7, s = (int)blockIdx.x >> 3, nbb = (P.B + RB - 1) / RB, S = P.S;
  if (bb >= nbb || (P.seats && s >= P.seats)) return;
  const int Hp = P.Hp, B = P.B, H = P.H, K = 4 * Hp;
  char* const stage = reinterpret_cast<char*>(lp_lds);
  float* const red = reinterpret_cast<float*>(stage + NM * SHARE);  // [2][NM][RB][PITCH]
  char* const ex = P.ex + (long)bb * S * BLK;                       // this block's images of the last step
  const long ex_step = (long)nbb * S * BLK;
  if (tid == 0) go_s[0] = go_s[1] = 1;
  if (wave == NM) {
    int local = 0;
    const int m = lx_meet(P.counters + bb * kLxSeats, S, s, lane, P.spin_limit, P.err, seat_s, local);
    if (lane == 0) seats_s = m, local_s = local;
  }
  // The UW columns of Wh' of a seat pass through LDS as they lie in memory, [gate row][unit]; the transposing reads
  // make the MFMA operands of them, which stay in registers.
  auto image = [&](int seat, int tid) {
    for (int i = tid; i < K * (UW / 8); i += 64 * (NM + 4)) {
      const int k = i / (UW / 8), x0 = (i - k * (UW / 8)) * 8, jj = seat * UW + x0;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (jj < Hp) v = *reinterpret_cast<const uint4*>(P.Wh + (long)k * Hp + jj);
      lp_lds[i] = v;
    }
    lp_barrier();
  };
  image(s, tid);
  const int seats = __builtin_amdgcn_readfirstlane(seats_s);
  if (seats <= 0) return;  // uniform
  if (wave < NM) {
    const int n = lane & 15, kg = lane >> 4;
    // slice q of the contraction, lane group kg: group of 8 units ug of gate `gate` of writer ws (the order of the images)
    Frag wf[KW][NB];
    const unsigned base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)lp_lds);
    auto weights = [&](int n, int kg) {
#pragma unroll
      for (int i = 0; i < KW; ++i) {
        const int g8 = (wave * KW + i) * 4 + kg, ws = g8 / (UW / 2), r8 = g8 - ws * (UW / 2), gate = r8 / (UW / 8), unit = ws * UW + (r8 - gate * (UW / 8)) * 8;
        const unsigned w = base + (unsigned)(((unit < Hp ? gate * Hp + unit : 0) + (n >> 2)) * (UW * 2) + (n & 3) * 8);
#pragma unroll
        for (int p = 0; p < NB; ++p) {
          if (p == 0) lds_read_tr16_b64<0>(wf[i][p].lo, w), lds_read_tr16_b64<4 * UW * 2>(wf[i][p].hi, w);
          else lds_read_tr16_b64<32>(wf[i][p].lo, w), lds_read_tr16_b64<4 * UW * 2 + 32>(wf[i][p].hi, w);
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int i = 0; i < KW; ++i) {
        const int g8 = (wave * KW + i) * 4 + kg, ws = g8 / (UW / 2), unit = ws * UW + ((g8 - ws * (UW / 2)) % (UW / 8)) * 8;
#pragma unroll
        for (int p = 0; p < NB; ++p) {
          frag_wait<false>(wf[i][p]);
          if (unit >= Hp) wf[i][p].lo = wf[i][p].hi = u32x2_t{0u, 0u};
        }
      }
      lp_barrier();
    };
    // operand of slice i in the share: writer i * 8 / UW of it (4 lane groups a slice, UW / 2 a writer)
    const char* op[NOFF];
#pragma unroll
    for (int o = 0; o < NOFF; ++o) {
      const int r8 = o * 4 + kg, gate = r8 / (UW / 8), ug = r8 - gate * (UW / 8);
      op[o] = stage + wave * SHARE + gate * GB + lx_at<RB>(n & (RB - 1), ug * 8);
    }
    const unsigned total = (unsigned)(S * BLK), share = (unsigned)(wave * SHARE);
    unsigned peek[1] = {share + (unsigned)((lane >> 3) * BLK)};
    peek[0] = (((lane >> 3) + 1) * BLK <= SHARE && peek[0] + BLK <= total ? peek[0] : 0u) + BLK - 128 + (lane & 7) * 16;
    const char* src = ex;  // images of the step before
    auto product = [&](int tt, int it) {
      if (tt > 0) {
        lp_u32x4 last[1];
        bool ok = lx_wait<1>(lp_buffer(src, total), peek, last, P.spin_limit, P.err);
        f32x4_t acc[NB][NA];
        for (long spins = 0; ok;) {
          // (every writer's last line is there, nearly always everything is: if not, the share is fetched again)
          unsigned l16 = (unsigned)lane * 16;
          if (UW == 24) asm volatile("" : "+v"(l16));  // (the addresses of all loads, kept from step to step, would spill)
#pragma unroll
          for (int i = 0; i < NL; ++i) {
            // What lies beyond the last writer is multiplied by zero weights, and 0 times an infinity or a NaN is a NaN: its
            // place in the operand of a row is filled from the same row, of the writers from the first on (24 units: 22 to
            // 32 of 32) or of the first writer (16: a load is one or two of its gates whole).
            const unsigned o = share + i * 1024, at = o + l16;
            const unsigned from = UW == 24 ? lx_min(at, at - total) : at < total ? at : l16;
            __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(src + from), ARD_LDS_PTR(stage + o), 16, 0, 16);
          }
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
          for (int p = 0; p < NB; ++p)
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[p][a][e] = 0.0f;
          unsigned most = 0;
          constexpr int GRP = KW > 8 ? 4 : KW;  // operands in registers at a time (12 and the weights of 24 units spill: 109 instead of 87 us, 8 rows)
#pragma unroll
          for (int i0 = 0; i0 < KW; i0 += GRP) {
            lp_u32x4 v[GRP];
#pragma unroll
            for (int k = 0; k < GRP; ++k) {
              const int i = i0 + k;
              v[k] = *reinterpret_cast<const lp_u32x4*>(op[i % NOFF] + (UW == 16 ? (i >> 1) * BLK + (i & 1) * 2 * GB : (i / 3) * BLK));
            }
#pragma unroll
            for (int k = 0; k < GRP; ++k) {
              const int i = i0 + k;
              most = lx_max3(lx_max3(most, v[k].x, v[k].y), v[k].z, v[k].w);
#pragma unroll
              for (int p = 0; p < NB; ++p)
                acc[p][i % NA] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, v[k]), frag_value<false>(wf[i][p]), acc[p][i % NA], 0, 0, 0);
            }
            if (GRP < KW) __builtin_amdgcn_sched_barrier(0);
          }
          if (!__any(most == kUnwritten)) break;
          ok = !lp_give_up(spins, P.spin_limit, P.err);
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        if (!ok) go_s[it & 1] = 0;
        else {
          // lane holds column n (unit), rows 4 kg + e
          float* const mine = red + ((it & 1) * NM + wave) * RB * PITCH;
#pragma unroll
          for (int p = 0; p < NB; ++p)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float x = acc[p][0][e] + acc[p][1][e];
              if constexpr (NA == 4) x += acc[p][2][e] + acc[p][3][e];
              if ((p == 0 || n < 8) && 4 * kg + e < RB) mine[(4 * kg + e) * PITCH + p * 16 + n] = x;
            }
        }
      }
      lp_barrier();
      return __builtin_amdgcn_readfirstlane(go_s[it & 1]) != 0;
    };
    weights(n, kg);
    for (int it = 0, tt = 0, i = 0; tt < P.T; ++it) {
      if (!product(tt, it)) return;
      if (++i == seats) i = 0, src += tt > 0 ? ex_step : 0, ++tt;
      if (seats > 1 && tt < P.T) {
        lp_barrier();  // (what the image overwrites has been read)
        const int l = lx_lane();
        image(__builtin_amdgcn_readfirstlane(seat_s[i]), wave * 64 + l);
        weights(l & 15, l >> 4);
      }
    }
    return;
  }
  const bool local = local_s != 0 && !P.spread;
  const int c0 = tid - 64 * NM;
  int row[NP], ul[NP], u[NP];
  unsigned at[NP], red_at[NP], c_at[NP], g_at[NP];  // byte of the cell's first word in the image; its place in a partial tile, in c, in the gates
  bool kept[NP], live[NP], in_store[NP];
  uint32_t mask[NP];  // all ones of a kept cell
  float dc_next[NP];
  auto cells = [&](int seat, int c0) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      lx_cell<RB>(p * 256 + c0, row[p], ul[p]);
      live[p] = p * 256 + c0 < RB * UW;
      at[p] = (unsigned)lx_at<RB>(row[p], ul[p]) & ~3u, red_at[p] = (unsigned)(row[p] * PITCH + ul[p]);
      const int j = seat * UW + ul[p], r = bb * RB + row[p];
      kept[p] = live[p] && j < P.Hk && r < B, in_store[p] = live[p] && j < Hp && r < B;
      u[p] = kept[p] ? P.off + j * P.step : 0;
      c_at[p] = (unsigned)(imin(r, B - 1) * H + u[p]), g_at[p] = (unsigned)(imin(r, B - 1) * 4 * H + u[p]);
      mask[p] = kept[p] ? ~0u : 0u;
      asm("" : "+v"(mask[p]));  // (or a branch comes of it)
      dc_next[p] = 0.0f;
    }
  };
  // what the cell of step t needs of the forward pass, fetched a step ahead (its c was the c_prev of the step before)
  float ni[NP], nf[NP], ng[NP], no[NP], nc[NP], np[NP];
  uint16_t nd[NP];
  auto fetch_cell = [&](int t) {
    const float* const ga = P.gates + (long)t * B * 4 * H;
    const float* const before = P.c + (long)(t > 0 ? t - 1 : 0) * B * H;
    const uint16_t* const dh = P.dh + (long)t * B * H;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      ni[p] = ga[g_at[p]], nf[p] = ga[g_at[p] + (unsigned)H], ng[p] = ga[g_at[p] + 2u * H], no[p] = ga[g_at[p] + 3u * H];
      nd[p] = dh[c_at[p]];
    }
    // (last: its copy waits for it, and so for all of them before the results are stored)
#pragma unroll
    for (int p = 0; p < NP; ++p) nc[p] = np[p], np[p] = before[c_at[p]];
  };
  auto fetch_first = [&](int t) {
#pragma unroll
    for (int p = 0; p < NP; ++p) np[p] = P.c[(long)t * B * H + c_at[p]];
    fetch_cell(t);
  };
  char* img = ex;  // images of the step
  auto cell = [&](int tt, int it, int seat, bool ahead) {
    const int t = P.T - 1 - tt;
    char* const out = img + seat * BLK;
    // all that does not depend on the gradient arriving from the step after, while the others are waited for:
    // d = (dc ki, dc kf, dc kg, dh ko) with dc = dh kc + dc_next
    float kc[NP], ki[NP], kf[NP], kg[NP], ko[NP], fg[NP], dh0[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const float gi = ni[p], gf = nf[p], gg = ng[p], go = no[p], cp = t > 0 ? np[p] : 0.0f, tc = lx_tanh(nc[p]);
      kc[p] = go * (1.0f - tc * tc), ki[p] = gg * gi * (1.0f - gi), kf[p] = cp * gf * (1.0f - gf), kg[p] = gi * (1.0f - gg * gg);
      ko[p] = tc * go * (1.0f - go), fg[p] = gf, dh0[p] = bf16_bits_to_f32(nd[p]);
      // (here: the compiler would do it, and wait for loads and stores, behind the barrier)
      asm volatile("" : "+v"(kc[p]), "+v"(ki[p]), "+v"(kf[p]), "+v"(kg[p]), "+v"(ko[p]), "+v"(fg[p]), "+v"(dh0[p]));
    }
    lp_barrier();
    if (!__builtin_amdgcn_readfirstlane(go_s[it & 1])) return false;
    unsigned word[NP][4];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (!live[p]) continue;
      float dh = dh0[p];
      if (tt > 0) {
        const float* src = red + (it & 1) * NM * RB * PITCH + red_at[p];
        float a[NM];
#pragma unroll
        for (int w = 0; w < NM; ++w) a[w] = src[w * RB * PITCH];
#pragma unroll
        for (int w = NM / 2; w > 0; w >>= 1)
#pragma unroll
          for (int i = 0; i < w; ++i) a[i] += a[i + w];
        dh += a[0];
      }
      const float dc = dh * kc[p] + dc_next[p];
      dc_next[p] = dc * fg[p];
      // dG_t to the other workgroups, then as the pass's result; padding units and rows store zeros
      const float d[4] = {dc * ki[p], dc * kf[p], dc * kg[p], dh * ko[p]};
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        word[p][g] = lx_word(__uint_as_float(__float_as_uint(d[g]) & mask[p]));
        if (!(c0 & 1)) lx_store(out, g * GB + at[p], word[p][g], local);
      }
    }
    if (ahead && t > 0) fetch_cell(t - 1);
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (!(c0 & 1) && in_store[p])
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<unsigned*>(P.dG + ((long)t * B + bb * RB + row[p]) * K + g * Hp + seat * UW + ul[p]) = word[p][g];
    return true;
  };
  cells(s, c0);
  fetch_first(P.T - 1);
  lp_barrier();
  for (int it = 0, tt = 0, i = 0, seat = s; tt < P.T; ++it) {
    if (!cell(tt, it, seat, seats == 1)) return;
    if (++i == seats) i = 0, ++tt, img += ex_step;
    if (seats > 1 && tt < P.T) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        if (kept[p]) P.dc[c_at[p]] = dc_next[p];
      seat = __builtin_amdgcn_readfirstlane(seat_s[i]);
      lp_barrier();
      const int l = lx_lane();
      image(seat, wave * 64 + l);
      lp_barrier();
      cells(seat, (wave - NM) * 64 + l);
      fetch_first(P.T - 1 - tt);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        if (tt > 0 && kept[p]) dc_next[p] = P.dc[c_at[p]];
      lx_landed();
    }
  }
}

}  // namespace ard
