// LSTM layer under a row pattern on its hidden units (Section 7.2.3: the LSTM runs as
// matrix multiplications, so the same patterns apply).
//
// Fused weight W[4H x (I+H)], gate blocks i, f, g, o of H rows, columns [x | h].
// A dropped unit has no gate rows and no recurrent column in any product.  Everything between
// the products lives in a COMPACT layout: Hk kept units stored with stride Hp = Hk rounded up
// to 8 (padding entries are zeros), gate g of kept unit j at index g*Hp + j.  All compact
// extents are then multiples of 8 and every product is a plain matrix product with 16-byte
// rows:
//   - the kept rows of the input and recurrent weights are gathered once per call
//     (Wx'[4Hp x I], Wh'[4Hp x Hp], zero rows / columns at the padding),
//   - the input projection of all T steps is one product, each step multiplies the compact
//     hidden state by Wh',
//   - the pointwise cell kernels run over physical units and write zeros for dropped ones,
//   - the weight gradient is computed compact and scattered into dW (zeros elsewhere) by one pass.
#include <stdlib.h>

#include <type_traits>

#include "fast.hpp"
#include "pattern.hpp"
#include "small.hpp"

namespace ard {

// Tile pattern over the fused weight W[4H x (I+H)] (Section 3.2): the synapse at (row, col) lies in tile
// (row / tr, col / tc), tiles are numbered row-major over a grid of `tcols` tile columns, and tile number
// t (0-based) is kept iff (t - o) mod dp == 0 (o = b - 1).  dp == 0: no tile pattern.
struct LstmTiles {
  int dp, o, tr, tc, tcols;
};
__device__ __forceinline__ bool lstm_synapse_kept(const LstmTiles& tp, int row, int col) {
  if (tp.dp <= 1) return true;
  const long t = (long)(row / tp.tr) * tp.tcols + col / tp.tc - tp.o;
  return t % tp.dp == 0;  // (sign of t is irrelevant for == 0)
}

// Eight consecutive elements from an address of any alignment, and the other way round
template <typename T> __device__ __forceinline__ void lstm_load8(const T* p, T (&v)[8]) {
  if ((((uintptr_t)p) & 15) == 0) {
#pragma unroll
    for (int i = 0; i < (int)sizeof(T) / 2; ++i) reinterpret_cast<uint4*>(v)[i] = reinterpret_cast<const uint4*>(p)[i];
  } else if ((((uintptr_t)p) & 3) == 0) {
#pragma unroll
    for (int i = 0; i < 2 * (int)sizeof(T); ++i) reinterpret_cast<uint32_t*>(v)[i] = reinterpret_cast<const uint32_t*>(p)[i];
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[i];
  }
}
template <typename T> __device__ __forceinline__ void lstm_store8(T* p, const T (&v)[8], int n) {
  if (n >= 8 && (((uintptr_t)p) & 15) == 0) {
#pragma unroll
    for (int i = 0; i < (int)sizeof(T) / 2; ++i) reinterpret_cast<uint4*>(p)[i] = reinterpret_cast<const uint4*>(v)[i];
  } else if (n >= 8 && (((uintptr_t)p) & 3) == 0) {
#pragma unroll
    for (int i = 0; i < 2 * (int)sizeof(T); ++i) reinterpret_cast<uint32_t*>(p)[i] = reinterpret_cast<const uint32_t*>(v)[i];
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < n) p[i] = v[i];
  }
}

// Kept units j .. j + 7 of the n of a row of them: every ax.step-th element of 8 ax.step, by 16-byte loads where the step is at most 4
// and another kept unit follows (the loads end before it), else one by one (n > j; those beyond n are not read, and zero).
template <typename T> __device__ __forceinline__ void lstm_gather8(const T* units, const Axis& ax, int j, T (&v)[8]) {
  if (ax.kind == AX_AFFINE && ax.step == 1 && j + 8 <= ax.n) return lstm_load8(units + ax.off + j, v);
  if constexpr (std::is_same<T, uint16_t>::value) {
    if (ax.kind == AX_AFFINE && ax.step <= 4 && j + 8 < ax.n) {
      auto wide = [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        SmallRaw<S> raw;
        small_load<S>(raw, units + ax.off + j * S, 0, 0);
        const bf16x8_t b = small_value<S>(raw);
        __builtin_memcpy(v, &b, 16);
      };
      if (ax.step == 2) wide(std::integral_constant<int, 2>{});
      else if (ax.step == 3) wide(std::integral_constant<int, 3>{});
      else wide(std::integral_constant<int, 4>{});
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = units[ax_phys(ax, imin(j + i, ax.n - 1))];
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (j + i >= ax.n) v[i] = (T)0;
}

// Everything a pass needs before its first product, in one launch (as five launches of a few microseconds each they
// took 33 us of a layer of 1500 units): eight consecutive elements of a row per thread.
template <typename T> struct LstmPrepare {
  Axis ax;
  int H, I, Ip, Hp;
  LstmTiles tp;
  // wxc[g*Hp + j][q] = W[(g*H + unit(j))][q], whc[g*Hp + j][q] = W[(g*H + unit(j))][I + unit(q)]; 0 at the padding and
  // for synapses of dropped tiles
  const T* W;
  T *wxc, *whc;
  const T* h;     // != NULL: hc[r][j] = h[r][unit(j)]
  T* hc;
  const T* x;     // != NULL: xp[r][q] = x[r][q], q < I, padded to Ip
  T* xp;
  int w0, w1, h0, h1, x0, x1;   // rows of each job that this launch takes
  int* rank;      // rank[u] = compact index of unit u or -1
  uint4* mark;    // exchange buffer of the recurrence: n16 pieces of kUnwritten
  long n16;
  int* sync;      // its status word and flags: zeros
  int n_sync;
  FastDiv by_cx, by_ch, by_hp;  // Ip / 8, Hp / 8, Hp
  int b_w, b_h, b_x, b_mark;    // workgroups of each job (the rank table takes one more)
};
constexpr unsigned kUnwritten = 0xffffffffu;
template <typename T> __global__ __launch_bounds__(256) void lstm_prepare_kernel(const LstmPrepare<T> P) {
  int b = (int)blockIdx.x;
  const int tid = threadIdx.x, cx = P.Ip >> 3, ch = P.Hp >> 3;
  T v[8];
  if (b < P.b_w) {
    const uint32_t e = (uint32_t)b * 256 + tid, nx = (uint32_t)(P.w1 - P.w0) * (uint32_t)cx;
    const bool rec = e >= nx;
    const uint32_t f = rec ? e - nx : e;
    const int rw = (int)fdiv(f, rec ? P.by_ch : P.by_cx), q = (int)(f - (uint32_t)rw * (uint32_t)(rec ? ch : cx)) * 8, r = P.w0 + rw;
    if (r >= P.w1) return;
    const int g = (int)fdiv((uint32_t)r, P.by_hp), j = r - g * P.Hp;
    const int prow = g * P.H + (j < P.ax.n ? ax_phys(P.ax, j) : 0);
    const T* row = P.W + (long)prow * (P.I + P.H);
    if (!rec && q + 8 <= P.I && P.tp.dp <= 1) {
      lstm_load8(row + q, v);
    } else if (rec && q < P.ax.n && P.tp.dp <= 1) {
      lstm_gather8(row + P.I, P.ax, q, v);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bool ok = rec ? q + i < P.ax.n : q + i < P.I;
        const int col = ok ? (rec ? P.I + ax_phys(P.ax, q + i) : q + i) : 0;
        v[i] = row[col];
        if (!ok || !lstm_synapse_kept(P.tp, prow, col)) v[i] = (T)0;
      }
    }
    if (j >= P.ax.n)
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = (T)0;
    return lstm_store8(rec ? P.whc + (long)r * P.Hp + q : P.wxc + (long)r * P.Ip + q, v, 8);
  }
  b -= P.b_w;
  if (b < P.b_h) {
    const uint32_t e = (uint32_t)b * 256 + tid;
    const uint32_t rh = fdiv(e, P.by_ch);
    const long r = P.h0 + (long)rh;
    if (r >= P.h1) return;
    const int j = (int)(e - rh * (uint32_t)ch) * 8;
    lstm_gather8(P.h + r * P.H, P.ax, j, v);
    return lstm_store8(P.hc + r * P.Hp + j, v, 8);
  }
  b -= P.b_h;
  if (b < P.b_x) {
    const uint32_t e = (uint32_t)b * 256 + tid;
    const uint32_t rx = fdiv(e, P.by_cx);
    const long r = P.x0 + (long)rx;
    if (r >= P.x1) return;
    const int q = (int)(e - rx * (uint32_t)cx) * 8;
    if (q + 8 <= P.I) {
      lstm_load8(P.x + r * P.I + q, v);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = q + i < P.I ? P.x[r * P.I + q + i] : (T)0;
    }
    return lstm_store8(P.xp + r * P.Ip + q, v, 8);
  }
  b -= P.b_x;
  if (b < P.b_mark) {
    const long i0 = (long)b * 256 + tid;
    if (i0 < P.n_sync) P.sync[i0] = 0;
    for (long i = i0; i < P.n16; i += (long)P.b_mark * 256) P.mark[i] = make_uint4(kUnwritten, kUnwritten, kUnwritten, kUnwritten);
    return;
  }
  for (int u = tid; u < P.H; u += 256) P.rank[u] = -1;
  __syncthreads();
  for (int j = tid; j < P.ax.n; j += 256) P.rank[ax_phys(P.ax, j)] = j;
}

__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + __expf(-z)); }

// One time step, forward.  G: compact pre-activations [B x 4Hp] (fp32).  Writes the
// activated gates [B x 4H], c [B x H] (fp32), h [B x H] (dtype) with zeros for dropped
// units, and the compact h [B x Hp] (zeros at the padding) that feeds the next step's product.
// Threads u >= H take the padding entries.
// `part` (optional): `splits` fp32 partial sums [B x 4Hp] of this step's recurrent product, `pstride`
// floats apart, added to G here (the product then needs no finishing pass).
template <typename T>
__global__ void lstm_cell_fwd_kernel(const float* G, const float* part, int splits, long pstride, const int* rank,
                                     const float* c_prev, int B, int H, int Hk, int Hp, float* gates, float* c, T* h,
                                     T* hc) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (u >= H) {
    const int j = Hk + (u - H);
    if (j < Hp) hc[(long)b * Hp + j] = (T)0;
    return;
  }
  const int j = rank[u];
  float gi = 0, gf = 0, gg = 0, go = 0, cv = 0, hv = 0;
  if (j >= 0) {
    const float* g = G + (long)b * 4 * Hp;
    float zi = g[j], zf = g[Hp + j], zg = g[2 * Hp + j], zo = g[3 * Hp + j];
    for (int s = 0; s < splits; ++s) {
      const float* q = part + s * pstride + (long)b * 4 * Hp;
      zi += q[j], zf += q[Hp + j], zg += q[2 * Hp + j], zo += q[3 * Hp + j];
    }
    gi = sigmoidf_(zi);
    gf = sigmoidf_(zf);
    gg = tanhf(zg);
    go = sigmoidf_(zo);
    const float cp = c_prev ? c_prev[(long)b * H + u] : 0.0f;
    cv = gf * cp + gi * gg;
    hv = go * tanhf(cv);
    hc[(long)b * Hp + j] = ElemTraits<T>::from_f32(hv);
  }
  float* ga = gates + (long)b * 4 * H;
  ga[u] = gi;
  ga[H + u] = gf;
  ga[2 * H + u] = gg;
  ga[3 * H + u] = go;
  c[(long)b * H + u] = cv;
  h[(long)b * H + u] = ElemTraits<T>::from_f32(hv);
}

// One time step, backward.  dh_next: compact [B x Hp] fp32 (NULL at the last step);
// dc_next: [B x H] fp32, read unless `first`, then overwritten.  Writes the compact gate
// gradient dG [B x 4Hp] in the storage dtype (zeros at the padding).
// dh_next may come as `splits` partial sums `pstride` floats apart (summed here).
template <typename T>
__global__ void lstm_cell_bwd_kernel(const float* gates, const float* c, const float* c_prev, const T* dh_ext,
                                     const float* dh_next, int splits, long pstride, float* dc_next, const int* rank, int B,
                                     int H, int Hk, int Hp, int first, T* dG) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  T* d = dG + (long)b * 4 * Hp;
  if (u >= H) {
    const int j = Hk + (u - H);
    if (j < Hp) d[j] = d[Hp + j] = d[2 * Hp + j] = d[3 * Hp + j] = (T)0;
    return;
  }
  const int j = rank[u];
  if (j < 0) return;
  const float* ga = gates + (long)b * 4 * H;
  const float gi = ga[u], gf = ga[H + u], gg = ga[2 * H + u], go = ga[3 * H + u];
  const float tc = tanhf(c[(long)b * H + u]);
  const float cp = c_prev ? c_prev[(long)b * H + u] : 0.0f;
  float dh = ElemTraits<T>::to_f32(dh_ext[(long)b * H + u]);
  if (dh_next)
    for (int s = 0; s < splits; ++s) dh += dh_next[s * pstride + (long)b * Hp + j];
  float dc = dh * go * (1.0f - tc * tc);
  if (!first) dc += dc_next[(long)b * H + u];
  d[j] = ElemTraits<T>::from_f32(dc * gg * gi * (1.0f - gi));
  d[Hp + j] = ElemTraits<T>::from_f32(dc * cp * gf * (1.0f - gf));
  d[2 * Hp + j] = ElemTraits<T>::from_f32(dc * gi * (1.0f - gg * gg));
  d[3 * Hp + j] = ElemTraits<T>::from_f32(dh * tc * go * (1.0f - go));
  dc_next[(long)b * H + u] = dc * gf;
}

// dst[r][0..cols) = src[r][0..cols) for rows of different lengths (ld_src, ld_dst): strips the padding of dx
template <typename T>
__global__ void lstm_copy_rows_kernel(const T* src, long ld_src, int cols, long ld_dst, T* dst) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const long r = blockIdx.y;
  if (j < cols) dst[r * ld_dst + j] = src[r * ld_src + j];
}

// dW[(g*H + u)][q] from the compact gradients dwx[4Hp x Ip] and dwh[4Hp x Hp]; +0.0 for every
// row of a dropped unit, every recurrent column of a dropped unit and every synapse of a dropped tile; gate rows p0 .. p1-1.
// The gradients come in the storage type, or (SUMS) as nx and nh fp32 partial sums of each, added in order and rounded once.
// Eight neighbouring columns of a row per thread (one at a time: 20 us where the bytes take 6, 512 of 1024 units); kept units in
// arithmetic progression are worked out, not looked up (LISTED), so that one load stands before the store, and those among
// eight recurrent columns are neighbours in the compact gradient: every second of 1500 units 19 -> 12 us.  (Four rows per thread
// took a fifth longer.)
struct LstmScatter {
  const void *x, *h;
  int nx, nh;
  Axis ax;  // kept units
  const int* rank;
  int H, I, Ip, Hp;
  LstmTiles tp;
  FastDiv by_chunks, by_h, by_step;
  int p0, p1;
  void* dW;
};
template <typename T, bool SUMS, bool LISTED>
__global__ __launch_bounds__(256) void lstm_scatter_dw_kernel(const LstmScatter P) {
  static_assert(!(SUMS && LISTED), "partial sums come from affine patterns");
  const uint32_t e = blockIdx.x * 256u + threadIdx.x;
  const int H = P.H, I = P.I, chunks = (I + H + 7) >> 3, row = (int)fdiv(e, P.by_chunks), q = (int)(e - (uint32_t)row * (uint32_t)chunks) * 8;
  const int p = P.p0 + row;  // physical gate row
  if (p >= P.p1) return;
  const int g = (int)fdiv((uint32_t)p, P.by_h), n = imin(8, I + H - q), u = p - g * H - P.ax.off, step = P.ax.step;
  const int j = LISTED ? P.rank[p - g * H] : u < 0 ? 0 : (int)fdiv((uint32_t)u, P.by_step);
  T v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (T)0;
  if (LISTED ? j >= 0 : u >= 0 && j * step == u && j < P.ax.n) {
    const long r = (long)g * P.Hp + j;
    if (q < I) {
      // (rows are padded to eight: beyond the input's last column lie zeros)
      if constexpr (SUMS) {
        const float* src = (const float*)P.x + r * P.Ip + q;
        const long plane = 4L * P.Hp * P.Ip;
        float s[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        for (int k = 0; k < P.nx; k += 2) {
          float4 t[4];
          const float4 *s0 = reinterpret_cast<const float4*>(src + k * plane), *s1 = reinterpret_cast<const float4*>(src + imin(k + 1, P.nx - 1) * plane);
          t[0] = s0[0], t[1] = s0[1], t[2] = s1[0], t[3] = s1[1];
          const float* f = reinterpret_cast<const float*>(t);
#pragma unroll
          for (int i = 0; i < 8; ++i) s[i] += f[i];
          if (k + 1 < P.nx)
#pragma unroll
            for (int i = 0; i < 8; ++i) s[i] += f[8 + i];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = ElemTraits<T>::from_f32(s[i]);
      } else {
        lstm_load8((const T*)P.x + r * P.Ip + q, v);
      }
    }
    if (LISTED && q + 8 > I) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = q + i - I, jv = c >= 0 && i < n ? P.rank[c] : -1;
        const T b = ((const T*)P.h)[r * P.Hp + (jv >= 0 ? jv : 0)];
        if (c >= 0) v[i] = jv >= 0 ? b : (T)0;
      }
    } else if (q + 8 > I) {
      // recurrent columns: kept unit j0 + t at column `at` of the eight
      const int c0 = q - I - P.ax.off, j0 = c0 <= 0 ? 0 : (int)fdiv((uint32_t)(c0 + step - 1), P.by_step);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (q + i >= I) v[i] = (T)0;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (t * step >= 8) break;
        const int jc = j0 + t, at = jc < P.ax.n ? jc * step - c0 : 8;
        const long from = r * P.Hp + imin(jc, P.Hp - 1);
        T b;
        if constexpr (SUMS) {
          const long plane = 4L * P.Hp * P.Hp;
          float s = 0.0f;
          for (int k = 0; k < P.nh; k += 4) {
            float f[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) f[i] = ((const float*)P.h)[imin(k + i, P.nh - 1) * plane + from];
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (k + i < P.nh) s += f[i];
          }
          b = ElemTraits<T>::from_f32(s);
        } else {
          b = ((const T*)P.h)[from];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = i == at ? b : v[i];
      }
    }
    if (P.tp.dp > 1)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (!lstm_synapse_kept(P.tp, p, q + i)) v[i] = (T)0;
  }
  lstm_store8((T*)P.dW + (long)p * (I + H) + q, v, n);
}

static bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// What workgroups exchange from step to step is its own flag: every word of the buffer holds kUnwritten when the
// kernel starts (no pair of bf16 results has these bits: f32_to_bf16_bits makes every NaN 0x7fc0), is written once
// with a device-scope store, and a reader takes its 16-byte pieces with device-scope loads until none holds the
// mark.  A step is then one store on its way to memory and one load that comes after it, where separate flags took
// four trips: the stores' acknowledgement, the flag's store, the poll and the load of the data.
typedef unsigned lp_u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bool lp_unwritten(const lp_u32x4& v) {
  return v.x == kUnwritten || v.y == kUnwritten || v.z == kUnwritten || v.w == kUnwritten;
}
// device-scope 16-byte load at byte `at` of the buffer (SC1: past the XCD's own caches)
__device__ __forceinline__ lp_u32x4 lp_load(__amdgpu_buffer_rsrc_t r, unsigned at) {
  return __builtin_bit_cast(lp_u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, 16));
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t lp_buffer(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}
// one more poll failed: true when this wavefront gives up
__device__ __forceinline__ bool lp_give_up(long& spins, long limit, int* err) {
  if (++spins <= limit && ((spins & 63) || !__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) return false;
  __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}
// ---- the recurrence in one launch (Section 7.2.3) -----------------------------------------------
//
// The per-step products of a batch-128 LSTM are a few hundred MFLOP each: issued as launches, a step
// costs two dependent launches however few units are kept.  This kernel walks all T steps itself.
// Workgroup (s, bb) owns 8 kept units (their 4 x 8 = 32 gate rows of Wh', staged ONCE in LDS for the whole
// sequence) and the MB = 32 * TMB batch rows of block bb: per step it multiplies h_{t-1}[rows, :] by its 32
// gate rows (32x32x16 MFMAs, the contraction dealt over the 4 wavefronts and summed through LDS), adds
// the input projection, runs the cell for its (row, unit) pairs (c stays in a register) and writes h_t.
// h_t travels between workgroups on different XCDs through device-scope (write-through) stores and device-scope
// loads that wait for the data itself (kUnwritten above).  Large states are read through L2 instead, with one flag per
// workgroup: after its h_t is written (its own stores waited for) a workgroup posts t + 1; a workgroup starts step t
// when the S workgroups of its batch block have all posted t.
// vmcnt counts loads and stores together and in order: what is not wanted by the next step (its outputs to the
// caller, two trips to memory) is stored, and the next step's projections are fetched, right after a wait has ended.  All workgroups must be resident together (the host launches this
// kernel only with at most one workgroup per CU); the wait is bounded all the same: a workgroup that gives
// up sets *err and leaves, and every workgroup that sees *err leaves too.
struct LstmPersist {
  const float* Gx;     // [T][B][4Hp] input projection
  const uint16_t* Wh;  // [4Hp][Hp] compact recurrent weight
  uint16_t* hc;        // [T][B][Hp] compact hidden states (written here, read by the next step)
  uint16_t* h;         // [T][B][H]
  float* c;            // [T][B][H]
  float* gates;        // [T][B][4H]
  int* counters;       // flags[batch block][unit slice] = steps posted by that workgroup, zero at launch
  int* err;            // zero at launch; 1: the recurrence gave up
  int T, B, H, Hk, Hp, S;
  int off, step;       // kept unit j is physical unit off + j * step
  long spin_limit;
  int spread;          // (a block per XCD) test hook: stores as if its workgroups were on several
  int seats;           // (the same) test hook: only so many workgroups of a block are there, 0: all
};

// VIA_L2: h_{t-1} is read through the XCD's L2 after an agent-scope acquire (else with device-scope loads)
// CH: 16-wide slices a wavefront has in flight
template <int TMB, bool VIA_L2, int CH>
__global__ __launch_bounds__(256) void lstm_persist_fwd_kernel(const LstmPersist P) {
  constexpr int MB = 32 * TMB;
  extern __shared__ uint4 lp_lds[];
  __shared__ int go_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int s = blockIdx.x % P.S, bb = blockIdx.x / P.S;
  const int Hp = P.Hp, B = P.B, H = P.H;
  const int pitch = Hp * 2 + 16;  // bytes between the staged weight rows (rows start 16 bytes apart in the banks)
  char* wl = reinterpret_cast<char*>(lp_lds);
  float* const reds = reinterpret_cast<float*>(wl + 32 * pitch);  // [TMB == 1 ? 2 : 1][4][MB][33]
  if (tid == 0) go_s = 1;
  // this workgroup's 32 gate rows, r = gate * 8 + local unit, staged once
  const int chunks = Hp >> 3;
  for (int i = tid; i < 32 * chunks; i += 256) {
    const int r = i / chunks, ch = i - r * chunks;
    const long row = (long)(r >> 3) * Hp + s * 8 + (r & 7);
    *reinterpret_cast<uint4*>(wl + r * pitch + ch * 16) = *reinterpret_cast<const uint4*>(P.Wh + row * Hp + ch * 8);
  }
  __syncthreads();
  const int nslice = (Hp + 15) >> 4;
  // cell: thread = (row rb of each 32-row tile, local unit ul)
  const int rb = tid >> 3, ul = tid & 7;
  const int j = s * 8 + ul;  // compact unit
  const bool kept = j < P.Hk;
  const int u = P.off + j * P.step;  // physical unit
  // zeros of the dropped units this thread owns: the rest of its group [j*step, (j+1)*step), the last kept
  // unit also the tail up to H
  const int z_lo = j * P.step, z_hi = !kept ? z_lo : (j == P.Hk - 1 ? H : z_lo + P.step);
  float c_reg[TMB];
#pragma unroll
  for (int rt = 0; rt < TMB; ++rt) c_reg[rt] = 0.0f;
  float zx[TMB][4];
  auto fetch_zx = [&](int t) {
    const float* Gt = P.Gx + (long)t * B * 4 * Hp;
#pragma unroll
    for (int rt = 0; rt < TMB; ++rt) {
      const int row = bb * MB + rt * 32 + rb;
#pragma unroll
      for (int g = 0; g < 4; ++g) zx[rt][g] = (row < B && kept) ? Gt[(long)row * 4 * Hp + g * Hp + j] : 0.0f;
    }
  };
  float gi[TMB], gf[TMB], gg[TMB], go[TMB], hv[TMB];
  auto store_outputs = [&](int t) {
#pragma unroll
    for (int rt = 0; rt < TMB; ++rt) {
      const int row = bb * MB + rt * 32 + rb;
      if (row >= B) continue;
      float* ga = P.gates + ((long)t * B + row) * 4 * H;
      if (kept) {
        ga[u] = gi[rt];
        ga[H + u] = gf[rt];
        ga[2 * H + u] = gg[rt];
        ga[3 * H + u] = go[rt];
        P.c[((long)t * B + row) * H + u] = c_reg[rt];
        P.h[((long)t * B + row) * H + u] = f32_to_bf16_bits(hv[rt]);
      }
      // zeros of the dropped units of this thread's group
      for (int uz = z_lo; uz < z_hi; ++uz) {
        if (uz == u) continue;
        ga[uz] = ga[H + uz] = ga[2 * H + uz] = ga[3 * H + uz] = 0.0f;
        P.c[((long)t * B + row) * H + uz] = 0.0f;
        P.h[((long)t * B + row) * H + uz] = 0;
      }
    }
  };
  if (!VIA_L2) fetch_zx(0);
  for (int t = 0; t < P.T; ++t) {
    float* const red = reds + (TMB == 1 ? (t & 1) * 4 * MB * 33 : 0);
    float zn[TMB][4];  // this step's projections
    f32x16_t acc[TMB];
#pragma unroll
    for (int rt = 0; rt < TMB; ++rt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[rt][v] = 0.0f;
    // this step's input projections do not depend on h_{t-1}: fetched before the wait, so that their
    // trip to memory overlaps it
    if (VIA_L2) fetch_zx(t);
#pragma unroll
    for (int rt = 0; rt < TMB; ++rt)
#pragma unroll
      for (int g = 0; g < 4; ++g) zn[rt][g] = zx[rt][g];
    if constexpr (!VIA_L2) {
      if (t > 0) {
        const auto hp = lp_buffer(P.hc + (long)(t - 1) * B * Hp, (unsigned)(B * Hp * 2));
        const int khalf = lane >> 5;
        unsigned rowb[TMB];
#pragma unroll
        for (int rt = 0; rt < TMB; ++rt) rowb[rt] = (unsigned)(imin(bb * MB + rt * 32 + (lane & 31), B - 1) * Hp * 2);  // (rows beyond the batch are never stored)
        bool gone = P.spin_limit < 0;  // (a negative bound is the host's way to force the give-up path)
        if (gone) __hip_atomic_store(P.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int q0 = wave; q0 < nslice && !gone; q0 += 4 * CH) {
          lp_u32x4 v[CH][TMB];
          long spins = 0;
          for (;;) {
            bool wait = false;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
              const int q = q0 + 4 * i, kk = q * 16 + khalf * 8;
              const int kc = (q < nslice && kk < Hp) ? kk : 0;  // (clamped: the value is discarded below)
#pragma unroll
              for (int rt = 0; rt < TMB; ++rt) v[i][rt] = lp_load(hp, rowb[rt] + kc * 2);
            }
#pragma unroll
            for (int i = 0; i < CH; ++i)
#pragma unroll
              for (int rt = 0; rt < TMB; ++rt) wait |= lp_unwritten(v[i][rt]);
            if (!__any(wait)) break;
            if ((gone = lp_give_up(spins, P.spin_limit, P.err))) break;
          }
          if (q0 == wave) {
            store_outputs(t - 1);
            if (t + 1 < P.T) fetch_zx(t + 1);
          }
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            const int q = q0 + 4 * i;
            if (q >= nslice) break;
            const int kk = q * 16 + khalf * 8;
            const bool k_ok = kk < Hp;
            const uint4 bw = *reinterpret_cast<const uint4*>(wl + (lane & 31) * pitch + (k_ok ? kk : 0) * 2);
            const bf16x8_t bfrag = __builtin_bit_cast(bf16x8_t, k_ok ? bw : make_uint4(0, 0, 0, 0));
#pragma unroll
            for (int rt = 0; rt < TMB; ++rt)
              acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, v[i][rt]), bfrag, acc[rt], 0, 0, 0);
          }
        }
        if (wave >= nslice) {  // (no slice: nothing to wait for)
          store_outputs(t - 1);
          if (t + 1 < P.T) fetch_zx(t + 1);
        }
        if (gone && lane == 0) go_s = 0;
      } else if (P.T > 1) {
        fetch_zx(1);
      }
    } else
    if (t > 0) {
      if (wave == 0) {
        // every workgroup of this batch block has posted step t - 1: one flag per workgroup (no contended
        // counter), the 64 lanes read 64 flags per poll
        const int* flags = P.counters + (long)bb * P.S;
        long spins = 0;
        int ok = 1;
        for (;;) {
          bool ready = true;
          for (int i = lane; i < P.S; i += 64) ready = ready && __hip_atomic_load(&flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= t;
          // (a negative bound is the host's way to force the give-up path: the first wait fails whatever it saw --
          // with a bound of zero a poll that finds everything posted, which is the common case, would still pass)
          if (__all(ready) && P.spin_limit >= 0) break;
          if (++spins > P.spin_limit || __hip_atomic_load(P.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            __hip_atomic_store(P.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = 0;
            break;
          }
        }
        if (lane == 0) go_s = ok;
        // (h_{t-1} is complete in memory: drop what this CU's L1 and this XCD's L2 may hold of it)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
      __syncthreads();
      if (!go_s) return;  // uniform: every thread of the workgroup leaves
      // recurrent product: this wavefront's 16-wide slices of the contraction
      const unsigned long long* hp = reinterpret_cast<const unsigned long long*>(P.hc + (long)(t - 1) * B * Hp);
      const int khalf = lane >> 5;
      // a wavefront issues the loads of CH slices together and multiplies afterwards (one round trip per CH slices
      // instead of one per slice)
      for (int q0 = wave; q0 < nslice; q0 += 4 * CH) {
        unsigned long long lo[CH][TMB], hi[CH][TMB];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int q = q0 + 4 * i;
          const int kk = q * 16 + khalf * 8;
          const int kc = (q < nslice && kk < Hp) ? kk : 0;  // (clamped: the value is discarded below)
#pragma unroll
          for (int rt = 0; rt < TMB; ++rt) {
            int row = bb * MB + rt * 32 + (lane & 31);
            row = row < B ? row : B - 1;  // rows beyond the batch are never stored
            const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(hp + (((long)row * Hp + kc) >> 2));
            lo[i][rt] = v.x, hi[i][rt] = v.y;
          }
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int q = q0 + 4 * i;
          if (q >= nslice) break;
          const int kk = q * 16 + khalf * 8;
          const bool k_ok = kk < Hp;
          const uint4 bw = *reinterpret_cast<const uint4*>(wl + (lane & 31) * pitch + (k_ok ? kk : 0) * 2);
          const bf16x8_t bfrag = __builtin_bit_cast(bf16x8_t, k_ok ? bw : make_uint4(0, 0, 0, 0));
#pragma unroll
          for (int rt = 0; rt < TMB; ++rt) {
            const uint4 aw = make_uint4((unsigned)lo[i][rt], (unsigned)(lo[i][rt] >> 32), (unsigned)hi[i][rt], (unsigned)(hi[i][rt] >> 32));
            acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, aw), bfrag, acc[rt], 0, 0, 0);
          }
        }
      }
    }
    // partial tiles of the four wavefronts -> LDS: lane holds column (lane & 31), rows 8*(v/4) + 4*(lane>>5) + v%4
#pragma unroll
    for (int rt = 0; rt < TMB; ++rt)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        red[(wave * MB + rt * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 33 + (lane & 31)] = acc[rt][v];
    __syncthreads();
    if (!go_s) return;  // uniform: every thread of the workgroup leaves
    // cell.  What the other workgroups wait for is h_t alone: it is stored first (device scope); gates, c and h go
    // to the caller's tensors off the critical path of the recurrence.
#pragma unroll
    for (int rt = 0; rt < TMB; ++rt) {
      const int rl = rt * 32 + rb, row = bb * MB + rl;
      hv[rt] = gi[rt] = gf[rt] = gg[rt] = go[rt] = 0.0f;
      if (row < B && kept) {
        float z[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int col = g * 8 + ul;
          z[g] = zn[rt][g] + ((red[(0 * MB + rl) * 33 + col] + red[(1 * MB + rl) * 33 + col]) +
                              (red[(2 * MB + rl) * 33 + col] + red[(3 * MB + rl) * 33 + col]));
        }
        gi[rt] = sigmoidf_(z[0]), gf[rt] = sigmoidf_(z[1]), gg[rt] = tanhf(z[2]), go[rt] = sigmoidf_(z[3]);
        const float cv = gf[rt] * c_reg[rt] + gi[rt] * gg[rt];
        c_reg[rt] = cv;
        hv[rt] = go[rt] * tanhf(cv);
      }
      if (row < B) {
        // compact h_t for the next step: device-scope store (the padding units store their zero)
        const unsigned bits = f32_to_bf16_bits(hv[rt]);
        const unsigned other = (unsigned)__shfl_xor((int)bits, 1, 64);
        if (!(ul & 1))
          __hip_atomic_store(reinterpret_cast<unsigned*>(P.hc + ((long)t * B + row) * Hp + j), bits | (other << 16), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (VIA_L2) {
      // every thread's h_t stores have completed before the workgroup signals
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0 && t + 1 < P.T)
        __hip_atomic_store(&P.counters[(long)bb * P.S + s], t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      store_outputs(t);
    } else if (TMB > 1) {
      __syncthreads();  // (one buffer of partial tiles: nobody overwrites it before everybody has read it)
    }
  }
  if (!VIA_L2) store_outputs(P.T - 1);
}

// ---- the backward recurrence in one launch ------------------------------------------------------
//
// Back-propagation through time has the same shape of problem: step t needs dG_{t+1} . Wh', the gradient
// that reaches h_t through the recurrence -- a contraction over all 4Hp gate rows (four times the forward
// one) for Hp outputs.  Workgroup (s, bb) owns UW kept units (16 or 32: their columns of Wh' are staged
// once in LDS, transposed) and MB = 16 * TM16 batch rows.  Per step it multiplies dG_{t+1}[rows, :] by its
// columns (16x16x32 MFMAs, the contraction dealt over the four wavefronts and summed through LDS), adds the
// gradient arriving at the output, runs the cell's backward for its (row, unit) pairs (the cell-state
// gradient stays in registers) and writes its 4 x UW columns of dG_t, which is the result and also what
// the other workgroups of the batch block wait for.  What a workgroup reads per step is MB x 4Hp values
// whatever UW is, so few rows per workgroup (and many workgroups) keep the step short.  Flags, scopes and
// the bounded wait are those of the forward kernel.
struct LstmPersistBwd {
  const float* gates;   // [T][B][4H]
  const float* c;       // [T][B][H]
  const uint16_t* dh;   // [T][B][H] gradient arriving at the outputs
  const uint16_t* Wh;   // [4Hp][Hp] compact recurrent weight
  uint16_t* dG;         // [T][B][4Hp] compact gate gradients
  int* counters;        // flags[batch block][unit slice] = steps posted by that workgroup, zero at launch
  int* err;             // zero at launch; 1: the recurrence gave up
  int T, B, H, Hk, Hp, S, UW;
  int off, step;        // kept unit j is physical unit off + j * step
  long spin_limit;
  char* ex;             // staging wavefronts, a block per XCD: [T][batch block][unit slice] blocks the workgroups exchange
  int spread, seats;    // as in LstmPersist
  float* dc;            // (a block per XCD) [B][H]: gradients of c, for workgroups that have several seats
};

template <int TM16, bool VIA_L2, int CH>
__global__ __launch_bounds__(256) void lstm_persist_bwd_kernel(const LstmPersistBwd P) {
  constexpr int MB = 16 * TM16;
  constexpr int NPMAX = 2 * TM16;  // (row, unit) pairs of a thread when UW = 32
  extern __shared__ uint4 lp_lds[];
  __shared__ int go_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int s = blockIdx.x % P.S, bb = blockIdx.x / P.S;
  const int Hp = P.Hp, B = P.B, H = P.H, UW = P.UW, K = 4 * Hp;
  const int pitch = K * 2 + 64;  // bytes between the staged columns (64 bytes apart in the banks)
  const int RW = UW + 1;
  char* wl = reinterpret_cast<char*>(lp_lds);
  float* const reds = reinterpret_cast<float*>(wl + UW * pitch);  // [VIA_L2 ? 1 : 2][4][MB][RW]
  if (tid == 0) go_s = 1;
  // this workgroup's UW columns of Wh', wl[local unit][gate row], staged once
  // (a row of Wh' is read in 16-byte pieces of 8 units: Hp and UW are multiples of 8)
  const int cpr = UW >> 3;
  for (int i = tid; i < K * cpr; i += 256) {
    const int k = i / cpr, x0 = (i - k * cpr) * 8;
    const int jj = s * UW + x0;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (jj < Hp) v = *reinterpret_cast<const uint4*>(P.Wh + (long)k * Hp + jj);
    const unsigned w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      *reinterpret_cast<uint16_t*>(wl + (x0 + e) * pitch + k * 2) = (uint16_t)(w4[e >> 1] >> ((e & 1) * 16));
  }
  __syncthreads();
  const int nslice = K >> 5;  // 32-deep slices (4Hp is a multiple of 32: no partial slice)
  const int nct = UW >> 4;    // 16-unit column tiles
  // cell: thread = (local unit ul, rows r0, r0 + rstep, ...)
  const int ul = tid % UW, r0 = tid / UW, rstep = 256 / UW, np = MB / rstep;
  const int j = s * UW + ul;  // compact unit
  const bool kept = j < P.Hk, in_store = j < Hp;
  const int u = kept ? P.off + j * P.step : 0;  // physical unit
  float dc_next[NPMAX];
#pragma unroll
  for (int i = 0; i < NPMAX; ++i) dc_next[i] = 0.0f;
  // what the cell of step t needs of the forward pass does not depend on the other workgroups: fetched a step ahead
  float ni[NPMAX], nf[NPMAX], ng[NPMAX], no[NPMAX], nc[NPMAX], np_c[NPMAX], nd[NPMAX];
  auto fetch_cell = [&](int t) {
#pragma unroll
    for (int i = 0; i < NPMAX; ++i) {
      ni[i] = nf[i] = ng[i] = no[i] = nc[i] = np_c[i] = nd[i] = 0.0f;
      const int row = bb * MB + r0 + i * rstep;
      if (i < np && row < B && kept) {
        const float* ga = P.gates + ((long)t * B + row) * 4 * H;
        ni[i] = ga[u], nf[i] = ga[H + u], ng[i] = ga[2 * H + u], no[i] = ga[3 * H + u];
        nc[i] = P.c[((long)t * B + row) * H + u];
        if (t > 0) np_c[i] = P.c[((long)(t - 1) * B + row) * H + u];
        nd[i] = bf16_bits_to_f32(P.dh[((long)t * B + row) * H + u]);
      }
    }
  };
  fetch_cell(P.T - 1);
  for (int tt = 0; tt < P.T; ++tt) {
    const int t = P.T - 1 - tt;
    float* const red = reds + (VIA_L2 ? 0 : (tt & 1) * 4 * MB * RW);
    if (VIA_L2 && tt > 0) fetch_cell(t);
    float gi[NPMAX], gf[NPMAX], gg[NPMAX], go[NPMAX], ct[NPMAX], cp[NPMAX], dhe[NPMAX];
#pragma unroll
    for (int i = 0; i < NPMAX; ++i)
      gi[i] = ni[i], gf[i] = nf[i], gg[i] = ng[i], go[i] = no[i], ct[i] = nc[i], cp[i] = np_c[i], dhe[i] = nd[i];
    f32x4_t acc[TM16][2];
#pragma unroll
    for (int rt = 0; rt < TM16; ++rt)
#pragma unroll
      for (int cti = 0; cti < 2; ++cti)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[rt][cti][v] = 0.0f;
    if constexpr (!VIA_L2) {
      if (tt > 0) {
        const auto gsrc = lp_buffer(P.dG + (long)(t + 1) * B * K, (unsigned)(B * K * 2));
        const int kgrp = lane >> 4, n = lane & 15;
        unsigned rowb[TM16];
#pragma unroll
        for (int rt = 0; rt < TM16; ++rt) rowb[rt] = (unsigned)(imin(bb * MB + rt * 16 + n, B - 1) * K * 2);  // (rows beyond the batch are never stored)
        bool gone = P.spin_limit < 0;  // (a negative bound is the host's way to force the give-up path)
        if (gone) __hip_atomic_store(P.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int q0 = wave; q0 < nslice && !gone; q0 += 4 * CH) {
          lp_u32x4 av[CH][TM16];
          long spins = 0;
          for (;;) {
            bool wait = false;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
              const int q = q0 + 4 * i, kc = q < nslice ? q * 32 + kgrp * 8 : 0;  // (clamped: the value is discarded below)
#pragma unroll
              for (int rt = 0; rt < TM16; ++rt) av[i][rt] = lp_load(gsrc, rowb[rt] + kc * 2);
            }
#pragma unroll
            for (int i = 0; i < CH; ++i)
#pragma unroll
              for (int rt = 0; rt < TM16; ++rt) wait |= lp_unwritten(av[i][rt]);
            if (!__any(wait)) break;
            if ((gone = lp_give_up(spins, P.spin_limit, P.err))) break;
          }
          if (q0 == wave && t > 0) fetch_cell(t - 1);
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            const int q = q0 + 4 * i;
            if (q >= nslice) break;
            const int kk = q * 32 + kgrp * 8;
#pragma unroll
            for (int cti = 0; cti < 2; ++cti) {
              if (cti >= nct) break;  // (uniform)
              const bf16x8_t bfrag = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(wl + (cti * 16 + n) * pitch + kk * 2));
#pragma unroll
              for (int rt = 0; rt < TM16; ++rt)
                acc[rt][cti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av[i][rt]), bfrag, acc[rt][cti], 0, 0, 0);
            }
          }
        }
        if (wave >= nslice && t > 0) fetch_cell(t - 1);  // (no slice: nothing to wait for)
        if (gone && lane == 0) go_s = 0;
      } else if (t > 0) {
        fetch_cell(t - 1);
      }
    } else if (tt > 0) {
      if (wave == 0) {
        // every workgroup of this batch block has posted dG_{t+1}
        const int* flags = P.counters + (long)bb * P.S;
        long spins = 0;
        int ok = 1;
        for (;;) {
          bool ready = true;
          for (int i = lane; i < P.S; i += 64) ready = ready && __hip_atomic_load(&flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= tt;
          if (__all(ready) && P.spin_limit >= 0) break;  // (a negative bound forces the give-up path)
          if (++spins > P.spin_limit || __hip_atomic_load(P.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            __hip_atomic_store(P.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = 0;
            break;
          }
        }
        if (lane == 0) go_s = ok;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
      __syncthreads();
      if (!go_s) return;  // uniform: every thread of the workgroup leaves
      const uint16_t* gsrc = P.dG + (long)(t + 1) * B * K;
      const int kgrp = lane >> 4, n = lane & 15;
      for (int q0 = wave; q0 < nslice; q0 += 4 * CH) {
        uint4 av[CH][TM16];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int q = q0 + 4 * i;
          const int kc = q < nslice ? q * 32 + kgrp * 8 : 0;  // (clamped: the value is discarded below)
#pragma unroll
          for (int rt = 0; rt < TM16; ++rt) {
            int row = bb * MB + rt * 16 + n;
            row = row < B ? row : B - 1;  // rows beyond the batch are never stored
            av[i][rt] = *reinterpret_cast<const uint4*>(gsrc + (long)row * K + kc);
          }
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int q = q0 + 4 * i;
          if (q >= nslice) break;
          const int kk = q * 32 + kgrp * 8;
#pragma unroll
          for (int cti = 0; cti < 2; ++cti) {
            if (cti >= nct) break;  // (uniform)
            const bf16x8_t bfrag = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(wl + (cti * 16 + n) * pitch + kk * 2));
#pragma unroll
            for (int rt = 0; rt < TM16; ++rt)
              acc[rt][cti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av[i][rt]), bfrag, acc[rt][cti], 0, 0, 0);
          }
        }
      }
    }
    // partial tiles of the four wavefronts -> LDS: lane holds column (lane & 15) of a tile, rows 4*(lane>>4) + v
#pragma unroll
    for (int rt = 0; rt < TM16; ++rt)
#pragma unroll
      for (int cti = 0; cti < 2; ++cti) {
        if (cti >= nct) break;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          red[(wave * MB + rt * 16 + 4 * (lane >> 4) + v) * RW + cti * 16 + (lane & 15)] = acc[rt][cti][v];
      }
    __syncthreads();
    if (!go_s) return;  // uniform: every thread of the workgroup leaves
#pragma unroll
    for (int i = 0; i < NPMAX; ++i) {
      if (i >= np) break;  // (uniform)
      const int rl = r0 + i * rstep, row = bb * MB + rl;
      float d[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (row < B && kept) {
        const float dh = dhe[i] + ((red[(0 * MB + rl) * RW + ul] + red[(1 * MB + rl) * RW + ul]) +
                                   (red[(2 * MB + rl) * RW + ul] + red[(3 * MB + rl) * RW + ul]));
        const float tc = tanhf(ct[i]);
        const float dc = dh * go[i] * (1.0f - tc * tc) + dc_next[i];
        d[0] = dc * gg[i] * gi[i] * (1.0f - gi[i]);
        d[1] = dc * cp[i] * gf[i] * (1.0f - gf[i]);
        d[2] = dc * gi[i] * (1.0f - gg[i] * gg[i]);
        d[3] = dh * tc * go[i] * (1.0f - go[i]);
        dc_next[i] = dc * gf[i];
      }
      // dG_t: pairs of adjacent units as one word, device-scope stores (the padding units store their zeros)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const unsigned bits = f32_to_bf16_bits(d[g]);
        const unsigned other = (unsigned)__shfl_xor((int)bits, 1, 64);
        if (!(ul & 1) && row < B && in_store)
          __hip_atomic_store(reinterpret_cast<unsigned*>(P.dG + ((long)t * B + row) * K + g * Hp + j), bits | (other << 16),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (VIA_L2) {
      // every thread's stores have completed before the workgroup signals
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0 && tt + 1 < P.T)
        __hip_atomic_store(&P.counters[(long)bb * P.S + s], tt + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---- both recurrences with staging wavefronts ---------------------------------------------------
//
// The recurrences below where a step's operands fit in LDS and the recurrent weights in registers (up to 1024 kept
// units): a workgroup has four wavefronts that compute and four that do nothing but fetch what the other workgroups
// write.  Measured in the kernels without them (512 kept units, B = 128): of 10300 clocks a step spent 5000 waiting
// for one round of device-scope loads that found everything written already, and 2400 between the loads and the
// product, issuing stores.  The loads took that long because
//  * a wavefront's MFMA operands are 32 bytes of each row, and a workgroup's results 16: every 128-byte line left
//    memory in four requests and came there in eight.  Here what a workgroup writes in a step is one contiguous
//    block in the order the fragments are read in, a store instruction is one whole line, and load instructions take
//    whole lines into LDS, from where the fragments come without bank conflicts;
//  * vmcnt counts a wavefront's stores and loads in one order: loads behind stores wait for their acknowledgement.
//    The fetching wavefronts store nothing.
// A step: fetch (loads until nothing in them is unwritten) | barrier | product, partial tiles to LDS | barrier | sum,
// cell, device-scope stores, the caller's outputs; the fetch of the next step starts at the second barrier.
// A step of 512 kept units, B = 128: forward 12700 -> 7550 clocks (waiting 3300 for the first line after its own cell,
// fetch 1740, product 710, cell 1300), backward 15600 -> 8230 (fetch 3350: 64 KB a workgroup); 64 steps 339 -> 203 us and
// 417 -> 225 us.  Starting the workgroups of an XCD at different lines, or more accumulators, changed nothing; 16-byte
// stores of single lanes instead of whole lines of words made the backward step 40 % longer.

// One wavefront's share of what the workgroups of a batch block wrote in a step: N KB at `at` + i KB of the block's
// `bytes` bytes, to `dst`.  First one line of every writer is polled past the caches (`peek`: the last it stores); when
// they have arrived, nearly always everything has, and the share is read through L2, where the workgroups of an XCD
// find what one of them fetched.  Only if a mark is left in it, a line was read too early and may lie in a cache: the
// share is then read past the caches until it is complete.  False: gave up.
template <int N, int NP>
__device__ __forceinline__ bool lp_fetch(const char* src, unsigned bytes, const unsigned (&at)[N], const unsigned (&peek)[NP], char* dst, int lane,
                                         long limit, int* err) {
  if (limit < 0) {  // (a negative bound is the host's way to force the give-up path)
    __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
  long spins = 0;
  const auto buf = lp_buffer(src, bytes);
  for (;;) {
    lp_u32x4 v[NP];
    bool wait = false;
#pragma unroll
    for (int i = 0; i < NP; ++i) v[i] = lp_load(buf, peek[i]);
#pragma unroll
    for (int i = 0; i < NP; ++i) wait |= lp_unwritten(v[i]);
    if (!__any(wait)) break;
    if (lp_give_up(spins, limit, err)) return false;
  }
  auto complete = [&] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bool wait = false;
#pragma unroll
    for (int i = 0; i < N; ++i) wait |= lp_unwritten(*reinterpret_cast<const lp_u32x4*>(dst + i * 1024 + lane * 16));
    return !__any(wait);
  };
#pragma unroll
  for (int i = 0; i < N; ++i) __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(src + at[i]), ARD_LDS_PTR(dst + i * 1024), 16, 0, 0);
  while (!complete()) {
    if (lp_give_up(spins, limit, err)) return false;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < N; ++i) __builtin_amdgcn_global_load_lds(ARD_GLB_PTR(src + at[i]), ARD_LDS_PTR(dst + i * 1024), 16, 0, 16);
  }
  return true;
}
// Workgroup -> (unit slice, batch block): XCD x = blockIdx % 8 takes the x-th eighth of the workgroups, batch block by
// batch block, so that an XCD fetches the rows of few batch blocks.
__device__ __forceinline__ bool lp_place(int S, int total, int& s, int& bb) {
  const int x = (int)blockIdx.x & 7, lo = (int)((long)x * total / 8), hi = (int)((long)(x + 1) * total / 8), L = lo + ((int)blockIdx.x >> 3);
  bb = L / S, s = L - bb * S;
  return L < hi;
}
__device__ __forceinline__ void lp_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  wg_barrier();
}

// Workgroup (s, bb): 8 * UT kept units, batch rows 32 bb .. 32 bb + 31.  KW: 16-wide slices of the contraction per wavefront.
template <int UT, int KW>
__global__ __launch_bounds__(512) void lstm_staged_fwd_kernel(const LstmPersist P) {
  constexpr int UW = 8 * UT, RP = 32 * UT + 1, BLK = 32 * UW * 2;  // BLK: bytes a workgroup writes in a step, [32 rows][UW units]
  extern __shared__ uint4 lp_lds[];
  __shared__ int go_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int s, bb;
  if (!lp_place(P.S, P.S * ((P.B + 31) / 32), s, bb)) return;
  const int Hp = P.Hp, B = P.B, H = P.H;
  char* const stage = reinterpret_cast<char*>(lp_lds);             // [4 KW] KB: blocks of the unit slices in order
  float* const red = reinterpret_cast<float*>(stage + 4096 * KW);  // [4][32][RP]
  char* const ex = reinterpret_cast<char*>(P.hc) + (long)bb * P.S * BLK;  // this batch block's blocks of step 0
  const long ex_step = (long)((B + 31) / 32) * P.S * BLK;
  if (tid == 0) go_s = 1;
  lp_barrier();
  if (wave >= 4) {
    const int w = wave - 4;
    const unsigned total = (unsigned)(P.S * BLK);
    unsigned at[KW], peek[1];
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      const unsigned o = (unsigned)((w * KW + i) * 1024 + lane * 16);
      at[i] = o < total ? o : (unsigned)(lane * 16) % BLK;  // (beyond the last slice: multiplied by zero weights)
    }
    {
      // the last line of slice `lane` of the share (a share is at most 32 slices; the rest look at its first one)
      const unsigned o = (unsigned)(w * KW * 1024 + (lane * BLK < KW * 1024 ? lane : 0) * BLK);
      peek[0] = (o < total ? o : 0u) + BLK - 128;
    }
    for (int t = 0; t < P.T; ++t) {
      if (t > 0 && !lp_fetch(ex + (t - 1) * ex_step, total, at, peek, stage + w * KW * 1024, lane, P.spin_limit, P.err)) go_s = 0;
      lp_barrier();
      if (!go_s) return;  // uniform: every wavefront reads it behind the same barrier
      lp_barrier();
    }
    return;
  }
  // this wavefront's part of the gate rows, in registers for the whole sequence: column r = gate * 8 + unit of tile ut
  const int khalf = lane >> 5, col = lane & 31;
  bf16x8_t wf[KW][UT];
#pragma unroll
  for (int i = 0; i < KW; ++i)
#pragma unroll
    for (int ut = 0; ut < UT; ++ut) {
      const int k = (wave * KW + i) * 16 + khalf * 8, unit = s * UW + ut * 8 + (col & 7);
      uint4 v = make_uint4(0, 0, 0, 0);
      if (k < Hp && unit < Hp) v = *reinterpret_cast<const uint4*>(P.Wh + ((long)(col >> 3) * Hp + unit) * Hp + k);
      wf[i][ut] = __builtin_bit_cast(bf16x8_t, v);
    }
  // cell: thread = (local unit ul, rows rb + i * 32 / UT)
  const int ul = tid % UW, rb = tid / UW;
  const int j = s * UW + ul;  // compact unit
  const bool kept = j < P.Hk;
  const int u = P.off + j * P.step;  // physical unit
  // zeros of the dropped units this thread owns: the rest of its group [j*step, (j+1)*step), the last kept
  // unit also the tail up to H
  const int z_lo = j * P.step, z_hi = !kept ? z_lo : (j == P.Hk - 1 ? H : z_lo + P.step);
  float c_reg[UT], zx[UT][4];
  auto fetch_zx = [&](int t) {
    const float* Gt = P.Gx + (long)t * B * 4 * Hp;
#pragma unroll
    for (int i = 0; i < UT; ++i) {
      const int row = imin(bb * 32 + rb + i * (32 / UT), B - 1), jj = imin(j, Hp - 1);  // (clamped: never used)
#pragma unroll
      for (int g = 0; g < 4; ++g) zx[i][g] = Gt[(long)row * 4 * Hp + g * Hp + jj];
    }
  };
#pragma unroll
  for (int i = 0; i < UT; ++i) c_reg[i] = 0.0f;
  fetch_zx(0);
  for (int t = 0; t < P.T; ++t) {
    lp_barrier();
    if (!go_s) return;
    f32x16_t acc[UT];
#pragma unroll
    for (int ut = 0; ut < UT; ++ut)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[ut][v] = 0.0f;
    if (t > 0) {
      const char* mine = stage + wave * KW * 1024;
      bf16x8_t af[KW];
#pragma unroll
      for (int i = 0; i < KW; ++i) af[i] = *reinterpret_cast<const bf16x8_t*>(mine + (UT == 1 ? (2 * i + khalf) * 32 + col : (i * 32 + col) * 2 + khalf) * 16);
#pragma unroll
      for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int ut = 0; ut < UT; ++ut) acc[ut] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], wf[i][ut], acc[ut], 0, 0, 0);
    }
    // partial tiles -> LDS: lane holds column (lane & 31), rows 8*(v/4) + 4*(lane>>5) + v%4
#pragma unroll
    for (int ut = 0; ut < UT; ++ut)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[(wave * 32 + 8 * (v >> 2) + 4 * khalf + (v & 3)) * RP + ut * 32 + col] = acc[ut][v];
    lp_barrier();
    // cell.  What the other workgroups wait for is h_t alone: it is stored first (device scope).
    unsigned* const mine = reinterpret_cast<unsigned*>(ex + t * ex_step + s * BLK);
    float gi[UT], gf[UT], gg[UT], go[UT], hv[UT];
#pragma unroll
    for (int i = 0; i < UT; ++i) {
      const int rl = rb + i * (32 / UT), row = bb * 32 + rl;
      float z[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int cl = (ul >> 3) * 32 + g * 8 + (ul & 7);
        z[g] = zx[i][g] + ((red[(0 * 32 + rl) * RP + cl] + red[(1 * 32 + rl) * RP + cl]) + (red[(2 * 32 + rl) * RP + cl] + red[(3 * 32 + rl) * RP + cl]));
      }
      gi[i] = sigmoidf_(z[0]), gf[i] = sigmoidf_(z[1]), gg[i] = tanhf(z[2]), go[i] = sigmoidf_(z[3]);
      const float cv = gf[i] * c_reg[i] + gi[i] * gg[i];
      c_reg[i] = cv;
      hv[i] = go[i] * tanhf(cv);
      const unsigned bits = kept ? f32_to_bf16_bits(hv[i]) : 0u;  // (the padding units store their zero)
      // (a wavefront's store is one whole line of the block; rows beyond the batch are stored like any other)
      const unsigned other = (unsigned)__shfl_xor((int)bits, 1, 64);
      if (!(ul & 1)) __hip_atomic_store(mine + (rl * UW + ul) / 2, bits | (other << 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (t + 1 < P.T) fetch_zx(t + 1);
#pragma unroll
    for (int i = 0; i < UT; ++i) {
      const int row = bb * 32 + rb + i * (32 / UT);
      if (row >= B) continue;
      float* ga = P.gates + ((long)t * B + row) * 4 * H;
      if (kept) {
        ga[u] = gi[i];
        ga[H + u] = gf[i];
        ga[2 * H + u] = gg[i];
        ga[3 * H + u] = go[i];
        P.c[((long)t * B + row) * H + u] = c_reg[i];
        P.h[((long)t * B + row) * H + u] = f32_to_bf16_bits(hv[i]);
      }
      for (int uz = z_lo; uz < z_hi; ++uz) {
        if (uz == u) continue;
        ga[uz] = ga[H + uz] = ga[2 * H + uz] = ga[3 * H + uz] = 0.0f;
        P.c[((long)t * B + row) * H + uz] = 0.0f;
        P.h[((long)t * B + row) * H + uz] = 0;
      }
    }
  }
}

// Workgroup (s, bb): 16 kept units, batch rows 16 bb .. 16 bb + 15.  KW: 32-wide slices of the contraction per wavefront.
template <int KW>
__global__ __launch_bounds__(512) void lstm_staged_bwd_kernel(const LstmPersistBwd P) {
  constexpr int BLK = 4 * 16 * 16 * 2;  // bytes a workgroup writes in a step, [4 gates][16 rows][16 units]
  extern __shared__ uint4 lp_lds[];
  __shared__ int go_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int s, bb;
  if (!lp_place(P.S, P.S * ((P.B + 15) / 16), s, bb)) return;
  const int Hp = P.Hp, B = P.B, H = P.H, K = 4 * Hp;
  char* const stage = reinterpret_cast<char*>(lp_lds);                    // [4 KW] KB: blocks of the unit slices in order
  float* const red = reinterpret_cast<float*>(stage + 4096 * KW + 1024);  // [4][16][17]
  char* const ex = P.ex + (long)bb * P.S * BLK;  // this batch block's blocks of step 0
  const long ex_step = (long)((B + 15) / 16) * P.S * BLK;
  // This workgroup's 16 columns of Wh', [unit][gate row], pass through LDS once (a row of Wh' is read in 16-byte
  // pieces of 8 units) and stay in registers.
  const int pitch = K * 2 + 64;  // (16 of them: at most 4096 KW + 1024 bytes)
  for (int i = tid; i < K * 2; i += 512) {
    const int k = i >> 1, x0 = (i & 1) * 8, jj = s * 16 + x0;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (jj < Hp) v = *reinterpret_cast<const uint4*>(P.Wh + (long)k * Hp + jj);
    const unsigned w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) *reinterpret_cast<uint16_t*>(stage + (x0 + e) * pitch + k * 2) = (uint16_t)(w4[e >> 1] >> ((e & 1) * 16));
  }
  if (tid == 0) go_s = 1;
  lp_barrier();
  const int kgrp = lane >> 4, n = lane & 15;
  // slice q of the contraction: units 16 (q / 2) + 8 (kgrp % 2) ... of gate 2 (q % 2) + kgrp / 2 (the order of the blocks)
  bf16x8_t wf[KW];
  if (wave < 4)
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      const int q = wave * KW + i, unit = (q >> 1) * 16 + (kgrp & 1) * 8;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (unit < Hp) v = *reinterpret_cast<const uint4*>(stage + n * pitch + ((2 * (q & 1) + (kgrp >> 1)) * Hp + unit) * 2);
      wf[i] = __builtin_bit_cast(bf16x8_t, v);
    }
  lp_barrier();
  if (wave >= 4) {
    const int w = wave - 4;
    const unsigned total = (unsigned)(P.S * BLK);
    unsigned at[KW], peek[1];
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      const unsigned o = (unsigned)((w * KW + i) * 1024 + lane * 16);
      at[i] = o < total ? o : (unsigned)(lane * 16);  // (beyond the last slice: multiplied by zero weights)
    }
    {
      const unsigned o = (unsigned)(w * KW * 1024 + (lane * BLK < KW * 1024 ? lane : 0) * BLK);
      peek[0] = (o < total ? o : 0u) + BLK - 128;
    }
    for (int tt = 0; tt < P.T; ++tt) {
      if (tt > 0 && !lp_fetch(ex + (tt - 1) * ex_step, total, at, peek, stage + w * KW * 1024, lane, P.spin_limit, P.err)) go_s = 0;
      lp_barrier();
      if (!go_s) return;
      lp_barrier();
    }
    return;
  }
  // cell: thread = (row tid / 16, local unit tid % 16)
  const int ul = tid & 15, rl = tid >> 4, row = bb * 16 + rl;
  const int j = s * 16 + ul;  // compact unit
  const bool kept = j < P.Hk && row < B, in_store = j < Hp && row < B;
  const int u = kept ? P.off + j * P.step : 0, rc = imin(row, B - 1);  // physical unit
  float dc_next = 0.0f;
  // what the cell of step t needs of the forward pass, fetched a step ahead
  float ni, nf, ng, no, nc, np, nd;
  auto fetch_cell = [&](int t) {
    const long at = (long)t * B + rc;
    const float* ga = P.gates + at * 4 * H;
    ni = ga[u], nf = ga[H + u], ng = ga[2 * H + u], no = ga[3 * H + u];
    nc = P.c[at * H + u];
    np = P.c[(at - (t > 0 ? B : 0)) * H + u];
    nd = bf16_bits_to_f32(P.dh[at * H + u]);
  };
  fetch_cell(P.T - 1);
  for (int tt = 0; tt < P.T; ++tt) {
    const int t = P.T - 1 - tt;
    lp_barrier();
    if (!go_s) return;
    f32x4_t acc[2];
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[0][v] = acc[1][v] = 0.0f;
    if (tt > 0) {
      const char* mine = stage + wave * KW * 1024 + (kgrp >> 1) * 512 + n * 32 + (kgrp & 1) * 16;
#pragma unroll
      for (int i = 0; i < KW; ++i) {
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(mine + i * 1024);
        acc[i & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wf[i], acc[i & 1], 0, 0, 0);
      }
    }
    // partial tiles -> LDS: lane holds column (lane & 15), rows 4*(lane>>4) + v
#pragma unroll
    for (int v = 0; v < 4; ++v) red[(wave * 16 + 4 * kgrp + v) * 17 + n] = acc[0][v] + acc[1][v];
    lp_barrier();
    const float gi = ni, gf = nf, gg = ng, go = no, ct = nc, cp = t > 0 ? np : 0.0f;
    float d[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (kept) {
      const float dh = nd + ((red[(0 * 16 + rl) * 17 + ul] + red[(1 * 16 + rl) * 17 + ul]) + (red[(2 * 16 + rl) * 17 + ul] + red[(3 * 16 + rl) * 17 + ul]));
      const float tc = tanhf(ct);
      const float dc = dh * go * (1.0f - tc * tc) + dc_next;
      d[0] = dc * gg * gi * (1.0f - gi);
      d[1] = dc * cp * gf * (1.0f - gf);
      d[2] = dc * gi * (1.0f - gg * gg);
      d[3] = dh * tc * go * (1.0f - go);
      dc_next = dc * gf;
    }
    // dG_t to the other workgroups (a wavefront's store is one whole line of the block), then as the pass's result;
    // padding units and rows store zeros
    unsigned* const mine = reinterpret_cast<unsigned*>(ex + tt * ex_step + s * BLK);
    unsigned word[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const unsigned bits = f32_to_bf16_bits(d[g]);
      word[g] = bits | ((unsigned)__shfl_xor((int)bits, 1, 64) << 16);
      if (!(ul & 1)) __hip_atomic_store(mine + ((g * 16 + rl) * 16 + ul) / 2, word[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (t > 0) fetch_cell(t - 1);
    if (!(ul & 1) && in_store)
#pragma unroll
      for (int g = 0; g < 4; ++g) *reinterpret_cast<unsigned*>(P.dG + ((long)t * B + row) * K + g * Hp + j) = word[g];
  }
}

}  // namespace ard

#include "lstm_xcd.hpp"
#include "lstm_step32.hpp"

namespace ard {

static int lstm_cu_count() {
  static int cus = -1;
  if (cus < 0) {
    int dev = 0;
    hipDeviceProp_t prop;
    cus = (!dry_run() && hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) ? prop.multiProcessorCount : 256;
  }
  return cus;
}

struct LstmWs {
  int* rank;
  char* wxc;     // [4Hp x Ip] dtype (Ip = I rounded up to 8: every row a whole number of 16-byte pieces)
  char* xp;      // [T*B x Ip] dtype, only when Ip != I: x with padded rows (forward, weight gradient)
  char* dxp;     // [T*B x Ip] dtype, only when Ip != I: dx before its padding is stripped
  char* whc;     // [4Hp x Hp] dtype
  char* hc;      // [T*B x Hp] dtype
  char* big;     // fwd: Gx [T*B x 4Hp] fp32; bwd: dG [T*B x 4Hp] dtype
  char* ex;      // (second half of big) bwd, bf16: blocks exchanged by the workgroups of the recurrence
  float* dh_next;  // [B x Hp]
  float* dc_next;  // [B x H]
  char* dwx;     // [4Hp x Ip] dtype
  char* dwh;     // [4Hp x Hp] dtype
  char* part;    // fp32 partial sums of split products
  size_t part_bytes;
  char *part_dwx, *part_dx;  // bf16: those of two products that run together with one whose sums are in `part` (fp32: `part`)
  size_t part_dwx_bytes, part_dx_bytes;
  int* sync;     // step counters (one per batch block of 32 rows) and the give-up flag of the one-launch recurrence
  size_t total;
};

static LstmWs lstm_ws_layout(char* base, int es, int T, int B, int I, int H, int Hk) {
  LstmWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align_up(bytes ? bytes : 1, 256);
    return p;
  };
  const size_t Hp = pad8(Hk);
  w.rank = (int*)take((size_t)H * 4);
  const size_t Ip = pad8(I);
  w.wxc = take(4 * Hp * Ip * es);
  w.xp = (int)Ip != I ? take((size_t)T * B * Ip * es) : nullptr;
  w.dxp = (int)Ip != I ? take((size_t)T * B * Ip * es) : nullptr;
  w.whc = take(4 * Hp * Hp * es);
  // (exchange blocks of the recurrences: whole blocks of 32 or 16 rows and 16 or 24 units)
  const size_t B32 = ((size_t)B + 31) / 32 * 32, B16 = ((size_t)B + 15) / 16 * 16, H24 = (Hp + 23) / 24 * 24;
  const size_t H16 = (Hp + 15) / 16 * 16 > H24 ? (Hp + 15) / 16 * 16 : H24;
  w.hc = take((size_t)T * B32 * H16 * es);
  w.big = take((size_t)T * B16 * 4 * H16 * 4);
  w.ex = w.big ? w.big + (size_t)T * B16 * 4 * H16 * 2 : nullptr;
  w.dh_next = (float*)take((size_t)B * Hp * 4);
  w.dc_next = (float*)take((size_t)B * H * 4);
  w.dwx = take(4 * Hp * Ip * es);
  w.dwh = take(4 * Hp * Hp * es);
  // room for the partial sums of any product here split 8 ways, capped at 256 MiB
  size_t big = 4 * Hp * (size_t)(Ip > Hp ? Ip : Hp);
  if ((size_t)B * 4 * Hp > big) big = (size_t)B * 4 * Hp;
  w.part_bytes = big * 4 * 8;
  if (w.part_bytes > ((size_t)256 << 20)) w.part_bytes = (size_t)256 << 20;
  w.part = take(w.part_bytes);
  w.part_dwx = w.part_dx = w.part, w.part_dwx_bytes = w.part_dx_bytes = w.part_bytes;
  if (es == 2) {  // (fp32 products run one after the other)
    w.part_dwx_bytes = split_part_bytes(4 * (long)Hp, (long)Ip), w.part_dx_bytes = split_part_bytes((long)T * B, (long)Ip);
    w.part_dwx = take(w.part_dwx_bytes), w.part_dx = take(w.part_dx_bytes);
  }
  w.sync = (int*)take(((size_t)pad8(Hk) / 8 * ((size_t)B / 32 + 1) + 8 + kLxBlocks * kLxSeats) * 4);
  w.total = off;
  return w;
}

struct LstmArgs {
  int32_t dtype, T, B, I, H, Hk, es;
  Axis ax;
  LstmTiles tiles;
};

static int32_t lstm_check(LstmArgs& a, const ard_pattern* pat) {
  if (a.dtype != ARD_F32 && a.dtype != ARD_BF16) return fail(ARD_EDTYPE, "unknown dtype %d", a.dtype);
  if (a.T <= 0 || a.B <= 0 || a.I <= 0 || a.H <= 0)
    return fail(ARD_ESHAPE, "T, B, I, H must be positive (got %d, %d, %d, %d)", a.T, a.B, a.I, a.H);
  if (4L * a.H > 65535) return fail(ARD_ESHAPE, "more than 16383 hidden units");
  a.tiles = LstmTiles{0, 0, 1, 1, 1};
  int32_t st;
  if (pat && pat->kind == ARD_PAT_TILE) {
    // synapses are dropped, every unit stays
    if (pat->tile_r <= 0 || pat->tile_c <= 0) return fail(ARD_EINVAL, "tile size must be positive");
    const int TR = ceil_div(4 * a.H, pat->tile_r), TC = ceil_div(a.I + a.H, pat->tile_c);
    st = check_pattern(pat, TR * TC, "pat");
    if (st) return st;
    a.tiles = LstmTiles{pat->dp, pat->b - 1, pat->tile_r, pat->tile_c, TC};
    a.ax = axis_identity(a.H);
  } else {
    st = check_pattern(pat, a.H, "pat");
    if (st) return st;
    a.ax = axis_of_pattern(pat, a.H);
  }
  a.Hk = a.ax.n;
  a.es = a.dtype == ARD_BF16 ? 2 : 4;
  if ((long)a.T * a.B > 0x7fffffffL / 4 || (long)a.B > 65535 || (long)a.T * a.B > 65535 * 64L)
    return fail(ARD_ESHAPE, "T*B or B too large");
  return ARD_OK;
}

// plain product C[M x N] (+)= A . B with identity maps on every side
static GemmParams plain_gemm(const void* A, long lda, const void* B, long ldb, void* C, long ldc, int M, int N, int K,
                             bool a_kc, bool b_kc, int ce, bool out_f32, float beta) {
  GemmParams P{};
  P.k = axis_identity(K);
  P.A = Operand{A, lda, axis_identity(M), 0, 0, 0, 0};
  P.B = Operand{B, ldb, axis_identity(N), 0, 0, 0, 0};
  P.A.vec = operand_vec_ok(P.A, a_kc, P.k, ce);
  P.B.vec = operand_vec_ok(P.B, b_kc, P.k, ce);
  P.C.p = C;
  P.C.ld = ldc;
  P.C.rm = axis_identity(M);
  P.C.cn = axis_identity(N);
  P.C.out_f32 = out_f32 ? 1 : 0;
  P.C.alpha = 1.0f;
  P.C.beta = beta;
  P.M = M;
  P.N = N;
  return P;
}

// Rows of `pieces` 8-element pieces that one job of a launch takes: a launch has less than 2^32 threads, one for each
// piece of its three jobs, and larger operands go in several.  (ARD_LSTM_PIECES: test hook, fewer pieces per job.)
static int lstm_rows_per_launch(long pieces) {
  const long most = getenv("ARD_LSTM_PIECES") ? atol(getenv("ARD_LSTM_PIECES")) : 1L << 30;
  const long rows = most / (pieces > 0 ? pieces : 1);
  return (int)(rows < 1 ? 1 : rows < 0x7fffffffL ? rows : 0x7fffffffL);
}
// What the recurrence of a pass wants cleared beforehand
struct LstmMark {
  void* buf;
  long bytes;
  int n_sync;
};
// Compact weights, padded x, (backward) compact h, rank table and marks; *xo: x with rows padded to a multiple of 8
// elements (zeros), so that the products over it can use 16-byte loads whatever the input width.
template <typename T>
static int32_t lstm_prepare(const LstmArgs& a, const void* W, const void* x, const void* h, const LstmMark& m, const LstmWs& w, hipStream_t stream,
                            const void** xo) {
  LstmPrepare<T> P{};
  P.ax = a.ax, P.H = a.H, P.I = a.I, P.Ip = pad8(a.I), P.Hp = pad8(a.Hk), P.tp = a.tiles;
  P.W = (const T*)W, P.wxc = (T*)w.wxc, P.whc = (T*)w.whc;
  P.h = (const T*)h, P.hc = (T*)w.hc;
  const bool pad = P.Ip != a.I;
  P.x = (const T*)x, P.xp = (T*)w.xp;
  *xo = pad ? (const void*)w.xp : x;
  P.rank = w.rank;
  P.mark = (uint4*)m.buf, P.n16 = m.bytes / 16, P.sync = w.sync, P.n_sync = m.n_sync;  // (exchange rows are whole pieces)
  const int cx = P.Ip / 8, ch = P.Hp / 8, rows = a.Hk > 0 ? a.T * a.B : 0;
  P.by_cx = fast_div((uint32_t)cx), P.by_ch = fast_div((uint32_t)ch), P.by_hp = fast_div((uint32_t)P.Hp);
  const long blocks = P.n16 || P.n_sync ? (P.n16 > P.n_sync ? P.n16 : P.n_sync) / 256 + 1 : 0;
  P.b_mark = (int)(blocks < 2048 ? blocks : 2048);
  const int nw = a.Hk > 0 ? 4 * P.Hp : 0, nh = h ? rows : 0, nx = pad ? rows : 0;
  const int step_w = lstm_rows_per_launch(cx + ch), step_h = lstm_rows_per_launch(ch), step_x = lstm_rows_per_launch(cx);
  do {
    P.w1 = nw - P.w0 < step_w ? nw : P.w0 + step_w, P.h1 = nh - P.h0 < step_h ? nh : P.h0 + step_h, P.x1 = nx - P.x0 < step_x ? nx : P.x0 + step_x;
    P.b_w = (int)(((long)(P.w1 - P.w0) * (cx + ch) + 255) / 256), P.b_h = (int)(((long)(P.h1 - P.h0) * ch + 255) / 256);
    P.b_x = (int)(((long)(P.x1 - P.x0) * cx + 255) / 256);
    ARD_LAUNCH(lstm_prepare_kernel<T>, dim3((unsigned)(P.b_w + P.b_h + P.b_x + P.b_mark + 1)), dim3(256), 0, stream, P);
    ARD_LAUNCH_CHECK("lstm_prepare_kernel");
    P.w0 = P.w1, P.h0 = P.h1, P.x0 = P.x1, P.b_mark = 0;
  } while (P.w0 < nw || P.h0 < nh || P.x0 < nx);
  return ARD_OK;
}

// An instance of a kernel in the record of a dry run: units per workgroup / 8, slices per wavefront
static const char* lstm_instance(const char* kernel, int ut, int kw) {
  static thread_local char name[64];
  snprintf(name, sizeof name, "%s %d %d", kernel, ut, kw);
  return name;
}

// The recurrences with staging wavefronts: kept units per workgroup (0: not taken).  One workgroup per CU, and as many
// of them as there are: narrow slices first.
static int lstm_staged_fwd_units(const LstmArgs& a) {
  const int Hp = pad8(a.Hk);
  if (a.dtype != ARD_BF16 || a.Hk <= 0 || a.T <= 1 || a.ax.kind != AX_AFFINE || getenv("ARD_NO_PERSIST") || Hp > 1024) return 0;
  for (int uw : {8, 16})
    if ((long)ceil_div(Hp, uw) * ceil_div(a.B, 32) <= lstm_cu_count()) return uw;
  return 0;
}
static bool lstm_staged_bwd(const LstmArgs& a) {
  const int Hp = pad8(a.Hk);
  return a.dtype == ARD_BF16 && a.Hk > 0 && a.T > 1 && a.ax.kind == AX_AFFINE && !getenv("ARD_NO_PERSIST") && Hp <= 1024 &&
         (long)ceil_div(Hp, 16) * ceil_div(a.B, 16) <= lstm_cu_count();
}

// The recurrences with a batch block per XCD: kept units per workgroup (0: not taken).  A block has at most the 32 CUs of
// an XCD, so the recurrent weights of its workgroups, in registers, end the range at 768 kept units, and eight blocks of
// 16 rows at a batch of 128.
static int lstm_xcd_units(const LstmArgs& a) {
  const int Hp = pad8(a.Hk);
  if (a.dtype != ARD_BF16 || a.Hk <= 0 || a.T <= 1 || a.ax.kind != AX_AFFINE || getenv("ARD_NO_PERSIST")) return 0;
  if (a.B > 16 * kLxBlocks || Hp > 24 * kLxSeats || lstm_cu_count() < kLxBlocks * kLxSeats) return 0;
  return Hp <= 16 * kLxSeats ? 16 : 24;
}

// Forward: two steps of more than 512 units are mostly start-up, which more, narrower workgroups all over the chip are
// through with sooner: staging wavefronts, 16.2 against 18.9 us (600 units, B = 1), 17.2 against 20.1 (B = 20), 21.8
// against 24.0 (680 units, B = 96), but 23.3 against 22.1 at B = 128.  Three steps are a draw: 21.5 against
// 25.0 (680 units, B = 32) to 31.2 against 29.2 (768, B = 96).
static int lstm_xcd_fwd_units(const LstmArgs& a) { return a.T == 2 && a.Hk > 512 && a.B <= 96 && lstm_staged_fwd_units(a) ? 0 : lstm_xcd_units(a); }
// Backward: 600 units, B = 128, 64 steps: 680 -> 400 us for the pass, 4 steps 81 -> 70.  Of two or three steps beyond the range
// of the staging wavefronts most is start-up (72 -> 65): they keep the form that still larger layers take.
static int lstm_xcd_bwd_units(const LstmArgs& a) { return lstm_staged_bwd(a) || a.T > 3 ? lstm_xcd_units(a) : 0; }
static int lstm_test_seats() { return getenv("ARD_LSTM_SEATS") ? atoi(getenv("ARD_LSTM_SEATS")) : 0; }
static int lstm_xcd_rows(int B) { return B <= 8 * kLxBlocks ? 8 : 16; }

// Does the forward pass of this layer run its recurrence in one launch, and how?  (bf16, affine pattern,
// at most one workgroup per CU, bounded exchange traffic)
struct PersistPlan {
  int tmb, S, nbb;
  int via_l2;  // read h_{t-1} through L2 (large states) instead of with device-scope loads
  size_t lds;
};
static bool lstm_persist_plan(const LstmArgs& a, PersistPlan& p) {
  const int Hp = pad8(a.Hk);
  if (a.dtype != ARD_BF16 || a.Hk <= 0 || a.T <= 1 || a.ax.kind != AX_AFFINE || getenv("ARD_NO_PERSIST")) return false;
  p.S = Hp / 8;
  p.tmb = 0;
  const int cus = lstm_cu_count();
  for (int cand = 1; cand <= 4 && !p.tmb; cand *= 2)
    if ((long)p.S * ceil_div(a.B, 32 * cand) <= cus) p.tmb = cand;
  if (!p.tmb) return false;
  p.nbb = ceil_div(a.B, 32 * p.tmb);
  // Every unit slice reads the whole h_{t-1} of its batch rows: S * B * Hp * 2 bytes per step over the chip.
  // Device-scope loads fetch each copy from the memory side: best while that volume is small (B = 128,
  // 512 kept units: 8 MB, 6.5 us per step against 12.6 for two launches per step), 15 us per step at 33 MB
  // (1024 units).  Larger states are read through the XCD's L2 after an agent-scope acquire, so the slices
  // of one XCD share one fetch: 12.8 us per step at 33 MB against 14.6 for launches, but 7.1 against 6.5 at
  // 8 MB (every workgroup's acquire drops what its neighbours just fetched).  Beyond 40 MB nothing was
  // measured: launch per step.
  const long traffic = (long)p.S * a.B * Hp * 2;
  p.via_l2 = traffic > (12L << 20);
  const bool traffic_ok = traffic <= (40L << 20);
  p.lds = (size_t)32 * (Hp * 2 + 16) + (size_t)4 * 32 * p.tmb * 33 * 4 * (p.tmb == 1 ? 2 : 1);
  return traffic_ok && p.lds <= 160 * 1024 - 1024;
}

struct PersistBwdPlan {
  int tm16, S, nbb, UW, via_l2;
  size_t lds;
};
// The backward recurrence in one launch.  Every unit slice reads the whole dG_{t+1} of its batch rows:
// S * B * 4Hp * 2 bytes per step over the chip, MB * 4Hp * 2 per workgroup.
static bool lstm_persist_bwd_plan(const LstmArgs& a, PersistBwdPlan& p) {
  const int Hp = pad8(a.Hk);
  if (a.dtype != ARD_BF16 || a.Hk <= 0 || a.T <= 1 || a.ax.kind != AX_AFFINE || getenv("ARD_NO_PERSIST")) return false;
  const int cus = lstm_cu_count();
  // Few rows and narrow slices first (most workgroups): at B = 128 with 512 kept units, per step of the whole
  // backward pass, 16 rows x 16 units (256 workgroups) 8.9 us, 16 x 32 10.4, 32 x 16 11.2, 32 x 32 13.6;
  // a launch per step 15.5.
  for (int tm = 1; tm <= 4; tm *= 2)
    for (int uw = 16; uw <= 32; uw *= 2) {
      const size_t lds = (size_t)uw * (8 * Hp + 64) + (size_t)4 * 16 * tm * (uw + 1) * 4 * 2;
      const int S = ceil_div(Hp, uw), nbb = ceil_div(a.B, 16 * tm);
      if (lds > 160 * 1024 - 1024 || (long)S * nbb > cus) continue;
      const long traffic = (long)S * a.B * 4 * Hp * 2;
      if (traffic > (40L << 20)) continue;
      // device-scope loads up to the volume they were measured best at (16 MB: 8.9 against 9.5 us through L2)
      p = PersistBwdPlan{tm, S, nbb, uw, traffic > (20L << 20), lds};
      return true;
    }
  return false;
}

// fp32: a launch per step that holds product and cell (else two).  Its tiles of 16 rows x 16 units read the weights once per
// 16 rows, which eats the launch it saves as layers grow: of 8 steps 1.3 to 1.8 times as fast up to 400 kept units and
// 120 rows, forward / backward 1.4 / 1.2 at 500 x 256, 1.2 / 1.1 at 22 x 878, 1.07 / 1.01 at 8 x 1334, 0.90 / 0.85 at 100 x 1300.
static bool lstm_step32(const LstmArgs& a) {
  return a.dtype == ARD_F32 && a.Hk > 0 && (long)ceil_div(a.B, 16) * a.Hk * a.Hk <= (1L << 21) && a.ax.kind == AX_AFFINE && a.ax.off < a.ax.step;
}

// (The forward kernel's threads write the zeros of their unit's dropped neighbours one after the other, which eats it where full tiles
// own units far apart: every eighth unit, 38 rows, 894 units, 8 steps 59 us with two launches a step and 77 with one, 8 rows, 626
// units 56 and 52.  Every sixth, 25 rows, 160 units 58 and 43, 17 rows, 1216 units 63 and 55.  One step alone has no product.)
static bool lstm_step32_fwd(const LstmArgs& a) {
  return lstm_step32(a) && a.T > 1 && (long)imin(a.B, 16) * imin(a.Hk, 16) * a.ax.step <= 1536;
}

template <typename T>
static int32_t lstm_fwd_t(const LstmArgs& a, const void* x, const void* W, void* h, float* c, float* gates,
                          const LstmWs& w, hipStream_t stream) {
  const int T_ = a.T, B = a.B, I = a.I, H = a.H, Hk = a.Hk, Hp = pad8(Hk), ce = 16 / a.es;
  // the whole recurrence in one launch when all of its workgroups fit on the chip together
  const int xcd = std::is_same<T, uint16_t>::value ? lstm_xcd_fwd_units(a) : 0, rb = lstm_xcd_rows(B);
  const int staged = !xcd && std::is_same<T, uint16_t>::value ? lstm_staged_fwd_units(a) : 0;
  PersistPlan pp;
  const bool persist = !xcd && !staged && std::is_same<T, uint16_t>::value && lstm_persist_plan(a, pp);
  LstmMark mark{};
  if (xcd) mark = LstmMark{w.hc, (long)(T_ - 1) * ceil_div(B, rb) * ceil_div(Hp, xcd) * rb * xcd * 2, 1 + kLxBlocks * kLxSeats};
  else if (staged) mark = LstmMark{w.hc, (long)(T_ - 1) * ceil_div(B, 32) * ceil_div(Hp, staged) * 64 * staged, 1};
  else if (persist) mark = LstmMark{w.hc, pp.via_l2 ? 0 : (long)(T_ - 1) * B * Hp * 2, pp.S * pp.nbb + 1};
  const void* xs;
  int32_t st = lstm_prepare<T>(a, W, x, nullptr, mark, w, stream, &xs);
  if (st) return st;
  float* Gx = (float*)w.big;
  const int Ip = pad8(I);
  if (Hk > 0) {
    // input projection of every step: Gx[T*B x 4Hp] = x . Wx'^T
    GemmParams P = plain_gemm(xs, Ip, w.wxc, Ip, Gx, 4 * Hp, T_ * B, 4 * Hp, Ip, true, true, ce, true, 0.0f);
    st = run_gemm(a.dtype, true, true, P, 0, 0, stream, w.part, w.part_bytes);
    if (st) return st;
  }
  if (xcd) {
    const int S = ceil_div(Hp, xcd);
    const long spin_limit = getenv("ARD_LSTM_SPIN_LIMIT") ? atol(getenv("ARD_LSTM_SPIN_LIMIT")) : 4000000L;
    LstmPersist P{Gx, (const uint16_t*)w.whc, (uint16_t*)w.hc, (uint16_t*)h, c, gates, w.sync + 1, w.sync, T_, B, H, Hk, Hp, S,
                  a.ax.off, a.ax.step, spin_limit, getenv("ARD_LSTM_SPREAD") ? 1 : 0, lstm_test_seats()};
    const int waves = lx_fwd_waves(xcd);
    const size_t lds = (size_t)2 * waves * rb * xcd * 16;
    auto launch = [&](auto kernel) -> int32_t {
      if (lds > 65536) ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, (int)lds));
      ARD_LAUNCH_NAMED("lstm_xcd_fwd_kernel", kernel, dim3((unsigned)(kLxBlocks * S)), dim3(64 * (waves + 4)), lds, stream, P);
      return ARD_OK;
    };
    if (rb == 8) st = xcd == 24 ? launch(lstm_xcd_fwd_kernel<8, 24, 3>) : Hp <= 256 ? launch(lstm_xcd_fwd_kernel<8, 16, 2>) : launch(lstm_xcd_fwd_kernel<8, 16, 4>);
    else st = xcd == 24 ? launch(lstm_xcd_fwd_kernel<16, 24, 3>) : Hp <= 256 ? launch(lstm_xcd_fwd_kernel<16, 16, 2>) : launch(lstm_xcd_fwd_kernel<16, 16, 4>);
    if (st) return st;
    ARD_LAUNCH_CHECK("lstm_xcd_fwd_kernel");
    return ARD_OK;
  }
  if (staged) {
    const int S = ceil_div(Hp, staged), kw = (int)align_up((size_t)ceil_div(Hp, 64), 4);
    const long spin_limit = getenv("ARD_LSTM_SPIN_LIMIT") ? atol(getenv("ARD_LSTM_SPIN_LIMIT")) : 4000000L;
    LstmPersist P{Gx, (const uint16_t*)w.whc, (uint16_t*)w.hc, (uint16_t*)h, c, gates, w.sync + 1, w.sync, T_, B, H, Hk, Hp, S,
                  a.ax.off, a.ax.step, spin_limit};
    const size_t lds = (size_t)4096 * kw + (size_t)4 * 32 * (4 * staged + 1) * 4;
    auto launch = [&](auto kernel) -> int32_t {
      if (lds > 65536) ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, (int)lds));
      ARD_LAUNCH_NAMED(lstm_instance("lstm_staged_fwd_kernel", staged / 8, kw), kernel, dim3((unsigned)(ceil_div(S * ceil_div(B, 32), 8) * 8)), dim3(512), lds, stream, P);
      return ARD_OK;
    };
    if (staged == 8) st = kw == 4 ? launch(lstm_staged_fwd_kernel<1, 4>) : kw == 8 ? launch(lstm_staged_fwd_kernel<1, 8>)
                          : kw == 12 ? launch(lstm_staged_fwd_kernel<1, 12>) : launch(lstm_staged_fwd_kernel<1, 16>);
    else st = kw == 4 ? launch(lstm_staged_fwd_kernel<2, 4>) : kw == 8 ? launch(lstm_staged_fwd_kernel<2, 8>)
              : kw == 12 ? launch(lstm_staged_fwd_kernel<2, 12>) : launch(lstm_staged_fwd_kernel<2, 16>);
    if (st) return st;
    ARD_LAUNCH_CHECK("lstm_staged_fwd_kernel");
    return ARD_OK;
  }
  if (persist) {
    const int S = pp.S, nbb = pp.nbb, tmb = pp.tmb;
    const size_t lds = pp.lds;
    // (ARD_LSTM_SPIN_LIMIT: test hook for the give-up path, negative = the first wait fails; a workgroup that
    // gives up leaves normally)
    const long spin_limit = getenv("ARD_LSTM_SPIN_LIMIT") ? atol(getenv("ARD_LSTM_SPIN_LIMIT")) : 4000000L;
    LstmPersist P{Gx, (const uint16_t*)w.whc, (uint16_t*)w.hc, (uint16_t*)h, c, gates, w.sync + 1, w.sync, T_, B, H, Hk, Hp, S,
                  a.ax.off, a.ax.step, spin_limit};
    const dim3 grid((unsigned)(S * nbb));
    auto launch = [&](auto kernel) -> int32_t {
      if (lds > 65536) ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, (int)lds));
      ARD_LAUNCH_NAMED("lstm_persist_fwd_kernel", kernel, grid, dim3(256), lds, stream, P);
      return ARD_OK;
    };
    // (tmb == 1: more than 1024 kept units, the staged kernel takes fewer)
    if (pp.via_l2) st = tmb == 1 ? launch(lstm_persist_fwd_kernel<1, true, 8>) : tmb == 2 ? launch(lstm_persist_fwd_kernel<2, true, 8>)
                                                                                             : launch(lstm_persist_fwd_kernel<4, true, 4>);
    else st = tmb == 1 ? launch(lstm_persist_fwd_kernel<1, false, 16>)
              : tmb == 2 ? launch(lstm_persist_fwd_kernel<2, false, 8>) : launch(lstm_persist_fwd_kernel<4, false, 4>);
    if (st) return st;
    ARD_LAUNCH_CHECK("lstm_persist_fwd_kernel");
    return ARD_OK;
  }
  if (lstm_step32_fwd(a)) {
    for (int t = 0; t < T_; ++t) {
      LstmStep32 P{};
      P.whc = (const float*)w.whc;
      P.G = Gx + (long)t * B * 4 * Hp;
      if (t > 0) P.hc_prev = (const float*)w.hc + (long)(t - 1) * B * Hp, P.c_prev = c + (long)(t - 1) * B * H;
      P.gates = gates + (long)t * B * 4 * H, P.c = c + (long)t * B * H, P.h = (float*)h + (long)t * B * H, P.hc = (float*)w.hc + (long)t * B * Hp;
      P.B = B, P.H = H, P.Hk = Hk, P.Hp = Hp, P.off = a.ax.off, P.step = a.ax.step;
      ARD_LAUNCH(lstm_step32_fwd_kernel, dim3(ceil_div(Hp, 16), ceil_div(B, 16)), dim3(64 * kStepWaves), 0, stream, P);
      ARD_LAUNCH_CHECK("lstm_step32_fwd_kernel");
    }
    return ARD_OK;
  }
  dim3 cgrid(ceil_div(H + (Hp - Hk), 256), B);
  for (int t = 0; t < T_; ++t) {
    float* Gt = Gx + (long)t * B * 4 * Hp;
    T* hc_t = (T*)w.hc + (long)t * B * Hp;
    int splits = 0;
    if (t > 0 && Hk > 0) {
      // recurrent part: G_t += h_{t-1}[kept] . Wh'^T, left as partial sums for the cell kernel when
      // the product runs on the LDS-direct kernels
      const T* hc_prev = (const T*)w.hc + (long)(t - 1) * B * Hp;
      GemmParams P = plain_gemm(hc_prev, Hp, w.whc, Hp, Gt, 4 * Hp, B, 4 * Hp, Hp, true, true, ce, true, 1.0f);
      if (run_gemm_partials(a.dtype, true, true, P, stream, w.part, w.part_bytes, &splits, &st)) {
        if (st) return st;
      } else {
        splits = 0;
        st = run_gemm(a.dtype, true, true, P, 0, 0, stream, w.part, w.part_bytes);
        if (st) return st;
      }
    }
    ARD_LAUNCH(lstm_cell_fwd_kernel<T>, cgrid, dim3(256), 0, stream, (const float*)Gt, (const float*)w.part, splits,
                       (long)B * 4 * Hp, (const int*)w.rank,
                       t > 0 ? (const float*)(c + (long)(t - 1) * B * H) : (const float*)nullptr, B, H, Hk, Hp,
                       gates + (long)t * B * 4 * H, c + (long)t * B * H, (T*)h + (long)t * B * H, hc_t);
    ARD_LAUNCH_CHECK("lstm_cell_fwd_kernel");
  }
  return ARD_OK;
}

// Weight gradients over many steps: tiles of 256 x 128 take less than half of the time per product that tiles of 64 x 64 take, but
// there are too few of them for the chip; split into partial sums, h and x of them, which the pass that spreads the gradients adds.
// Both ways cost, in us at 256 CUs: the launch that small tiles share, 8.4 and per step of a CU's 64 x 64 (128 x 64) tiles 0.237 (0.39),
// the gradient of x among them where its tiles are 64 x 64, which else has a launch of its own; large tiles 4.6 a launch, 7.2 a round,
// 0.57 to 0.815 a step the fuller the round; each MB of partial sums 0.04 to read, beyond 89 MB 0.37, and those of the recurrent
// columns, a kept unit at a time, 0.77 per MB of the gradient for every four of them.  Fitted to the kernels of 170 layers (1024 -
// 16384 rows, I and H 256 - 2048, dp 1 - 4), large tiles to 3 %, the others to 10 %; in whole backward passes, where three launches take
// the place of one, the large tiles cost 10 us more than their kernels (100 layers).  Over 220 other layers, backward pass, 0.997 of the time of
// the former estimate, none slower than with small tiles alone.  The line: backward passes in us with
// small tiles and with partial sums, T = 24, B = 115, I = 900, H = 1529, dp = 2 197 and 209, 92, 48, 1280, 1088, 2 302 and 314, 24, 128, 801, 801, 1
// 413 and 420, none of them taken; 36, 101, 768, 1675, 2 522 and 517, 78, 64, 1000, 1408, 2 349 and 336, 60, 128, 1024, 1024, 2 288 and 283,
// 64, 128, 960, 960, 2 295 and 284, 85, 88, 1032, 1280, 2 554 and 494, all taken.  Where the recurrent weight's large tiles
// fill the chip by themselves, summing their kept columns costs more than it gives (120, 83, 256, 1696, 1 2507 and 2545).
static bool lstm_sum_splits(const LstmArgs& a, int Ip, int Hp, size_t room, int& h, int& x) {
  h = x = 0;
  if (a.dtype != ARD_BF16 || a.T < 2 || a.ax.kind != AX_AFFINE || dev_knobs().no_fast) return false;
  const int rows = a.T * a.B, rows_h = rows - a.B, M = 4 * Hp;
  // what a product of 4-wavefront tiles adds to the launch they share (-1: it has larger ones)
  auto share = [](int m, int n, int k, bool tall) {
    if ((long)ceil_div(m, 256) * ceil_div(n, 128) >= 220 || (long)ceil_div(m, 128) * ceil_div(n, 128) >= 440) return -1.0f;
    const float steps = ceil_div(k, 64) / 256.0f;
    if ((long)ceil_div(m, 128) * ceil_div(n, 64) >= 440) return tall ? 0.39f * ceil_div(m, 128) * ceil_div(n, 64) * steps : -1.0f;
    return 0.237f * ceil_div(m, 64) * ceil_div(n, 64) * steps;
  };
  auto large = [&](int n, int k, int splits) {
    const int tiles = ceil_div(M, 256) * ceil_div(n, 128) * splits, steps = ceil_div(ceil_div(k, 64), splits);
    const float last = (tiles % 256) / 256.0f;
    return 4.6f + tiles / 256 * (0.815f * steps + 7.2f) + (last > 0 ? (0.57f + 0.245f * last) * steps + 7.2f * fmaxf(last, 0.6f) : 0.0f);
  };
  const float small_x = share(M, Ip, rows, true), small_h = share(M, Hp, rows_h, true), dx = share(rows, Ip, M, false);
  if (small_h < 0) return false;
  const float small = 8.4f + (small_x < 0 ? large(Ip, rows, 1) : small_x) + small_h + (dx < 0 ? 0.0f : dx);
  const float alone = 10.0f + (dx < 0 ? 0.0f : 6.5f + 0.8f * dx);
  float best = small;
  for (int sx = 1; sx <= 8 && sx * 4 <= ceil_div(rows, 64); ++sx)
    for (int sh = 1; sh <= 8 && sh * 4 <= ceil_div(rows_h, 64); ++sh) {
      const size_t bytes = (size_t)16 * Hp * ((size_t)sx * Ip + (size_t)sh * Hp);
      if (bytes > room) break;
      const float mb = bytes * 1e-6f, spread = 0.04f * mb + 0.33f * fmaxf(mb - 89.0f, 0.0f) + 0.77f * 16e-6f * Hp * Hp * ceil_div(sh, 4);
      const float t = large(Ip, rows, sx) + large(Hp, rows_h, sh) + alone + spread;
      if (t < best) best = t, x = sx, h = sh;
    }
  return x > 0;
}

template <typename T>
static int32_t lstm_bwd_t(const LstmArgs& a, const void* x, const void* W, const void* h, const float* c,
                          const float* gates, const void* dh, void* dx, void* dW, const LstmWs& w,
                          hipStream_t stream) {
  const int T_ = a.T, B = a.B, I = a.I, H = a.H, Hk = a.Hk, Hp = pad8(Hk), ce = 16 / a.es;
  const int Ip = pad8(I);
  if (Hk == 0) {
    if (int32_t st = fill_matrix(a.dtype, dx, (long)T_ * B * I, 0.0f, stream)) return st;
    return fill_matrix(a.dtype, dW, (long)4 * H * (I + H), 0.0f, stream);
  }
  PersistBwdPlan bp;
  const int xcd = std::is_same<T, uint16_t>::value ? lstm_xcd_bwd_units(a) : 0, rb = lstm_xcd_rows(B);
  const bool staged = std::is_same<T, uint16_t>::value && lstm_staged_bwd(a);
  const bool one_launch = xcd || staged || (std::is_same<T, uint16_t>::value && lstm_persist_bwd_plan(a, bp));
  const long step_bytes = (long)B * 4 * Hp * 2;
  LstmMark mark{};  // (dG_0 is waited for by nobody)
  if (xcd) mark = LstmMark{w.ex, (long)(T_ - 1) * ceil_div(B, rb) * ceil_div(Hp, xcd) * rb * xcd * 8, 1 + kLxBlocks * kLxSeats};
  else if (staged) mark = LstmMark{w.ex, (long)(T_ - 1) * ceil_div(B, 16) * ceil_div(Hp, 16) * 2048, 1};
  else if (one_launch) mark = LstmMark{w.big + step_bytes, bp.via_l2 ? 0 : (T_ - 1) * step_bytes, bp.S * bp.nbb + 1};
  // (hc: compact copy of the stored hidden states, h[:, kept])
  const void* xs;
  int32_t st = lstm_prepare<T>(a, W, x, h, mark, w, stream, &xs);
  if (st) return st;
  T* dG = (T*)w.big;
  dim3 cgrid(ceil_div(H + (Hp - Hk), 256), B);
  const float* dh_src = nullptr;  // dh_t[kept] from the product of step t+1: partial sums or w.dh_next
  int dh_splits = 0;
  if (xcd) {
    const int S = ceil_div(Hp, xcd), kw = xcd == 24 ? 12 : S <= 8 ? 2 : S <= 16 ? 4 : 8;
    const long spin_limit = getenv("ARD_LSTM_SPIN_LIMIT") ? atol(getenv("ARD_LSTM_SPIN_LIMIT")) : 4000000L;
    LstmPersistBwd P{gates, c, (const uint16_t*)dh, (const uint16_t*)w.whc, (uint16_t*)dG, w.sync + 1, w.sync, T_, B, H, Hk, Hp,
                     S, xcd, a.ax.off, a.ax.step, spin_limit, w.ex, getenv("ARD_LSTM_SPREAD") ? 1 : 0, lstm_test_seats(), w.dc_next};
    const size_t image = (size_t)4 * Hp * xcd * 2 + 64, step = kLxBwdWaves * ((size_t)kw * rb * 64 + (size_t)2 * rb * (xcd + 4) * 4);
    const size_t lds = image > step ? image : step;
    auto launch = [&](auto kernel) -> int32_t {
      if (lds > 65536) ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, (int)lds));
      ARD_LAUNCH_NAMED("lstm_xcd_bwd_kernel", kernel, dim3((unsigned)(kLxBlocks * S)), dim3(64 * (kLxBwdWaves + 4)), lds, stream, P);
      return ARD_OK;
    };
    if (rb == 8) st = kw == 12 ? launch(lstm_xcd_bwd_kernel<8, 24, 12>) : kw == 8 ? launch(lstm_xcd_bwd_kernel<8, 16, 8>)
                      : kw == 4 ? launch(lstm_xcd_bwd_kernel<8, 16, 4>) : launch(lstm_xcd_bwd_kernel<8, 16, 2>);
    else st = kw == 12 ? launch(lstm_xcd_bwd_kernel<16, 24, 12>) : kw == 8 ? launch(lstm_xcd_bwd_kernel<16, 16, 8>)
              : kw == 4 ? launch(lstm_xcd_bwd_kernel<16, 16, 4>) : launch(lstm_xcd_bwd_kernel<16, 16, 2>);
    if (st) return st;
    ARD_LAUNCH_CHECK("lstm_xcd_bwd_kernel");
  } else if (staged) {
    // (17 to 24 slices: with 256 CUs the recurrences with a block per XCD take all such layers)
    const int S = ceil_div(Hp, 16), need = ceil_div(Hp, 32), kw = need <= 4 ? 4 : need <= 8 ? 8 : need <= 16 ? 16 : 32;
    const long spin_limit = getenv("ARD_LSTM_SPIN_LIMIT") ? atol(getenv("ARD_LSTM_SPIN_LIMIT")) : 4000000L;
    LstmPersistBwd P{gates, c, (const uint16_t*)dh, (const uint16_t*)w.whc, (uint16_t*)dG, w.sync + 1, w.sync, T_, B, H, Hk, Hp,
                     S, 16, a.ax.off, a.ax.step, spin_limit, w.ex};
    const size_t lds = (size_t)4096 * kw + 1024 + (size_t)4 * 16 * 17 * 4;
    auto launch = [&](auto kernel) -> int32_t {
      if (lds > 65536) ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, (int)lds));
      ARD_LAUNCH_NAMED(lstm_instance("lstm_staged_bwd_kernel", 2, kw), kernel, dim3((unsigned)(ceil_div(S * ceil_div(B, 16), 8) * 8)), dim3(512), lds, stream, P);
      return ARD_OK;
    };
    st = kw == 4 ? launch(lstm_staged_bwd_kernel<4>) : kw == 8 ? launch(lstm_staged_bwd_kernel<8>)
         : kw == 16 ? launch(lstm_staged_bwd_kernel<16>) : launch(lstm_staged_bwd_kernel<32>);
    if (st) return st;
    ARD_LAUNCH_CHECK("lstm_staged_bwd_kernel");
  } else if (one_launch) {
    const long spin_limit = getenv("ARD_LSTM_SPIN_LIMIT") ? atol(getenv("ARD_LSTM_SPIN_LIMIT")) : 4000000L;
    LstmPersistBwd P{gates, c, (const uint16_t*)dh, (const uint16_t*)w.whc, (uint16_t*)dG, w.sync + 1, w.sync, T_, B, H, Hk, Hp,
                     bp.S, bp.UW, a.ax.off, a.ax.step, spin_limit};
    const dim3 grid((unsigned)(bp.S * bp.nbb));
    const size_t lds = bp.lds;
    auto launch = [&](auto kernel) -> int32_t {
      if (lds > 65536) ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, (int)lds));
      ARD_LAUNCH_NAMED("lstm_persist_bwd_kernel", kernel, grid, dim3(256), lds, stream, P);
      return ARD_OK;
    };
    const bool deep = Hp > 512;  // (slices of a wavefront: one round trip for up to 1024 kept units)
    if (bp.via_l2) st = bp.tm16 == 1 ? launch(lstm_persist_bwd_kernel<1, true, 16>) : bp.tm16 == 2 ? launch(lstm_persist_bwd_kernel<2, true, 8>)
                                                                                                 : launch(lstm_persist_bwd_kernel<4, true, 4>);
    else st = bp.tm16 == 1 ? (deep ? launch(lstm_persist_bwd_kernel<1, false, 32>) : launch(lstm_persist_bwd_kernel<1, false, 16>))
              : bp.tm16 == 2 ? launch(lstm_persist_bwd_kernel<2, false, 8>) : launch(lstm_persist_bwd_kernel<4, false, 4>);
    if (st) return st;
    ARD_LAUNCH_CHECK("lstm_persist_bwd_kernel");
  }
  const bool step32 = lstm_step32(a);
  for (int t = step32 ? T_ - 1 : -1; t >= 0; --t) {
    LstmStep32 P{};
    P.whc = (const float*)w.whc;
    P.gates = const_cast<float*>(gates) + (long)t * B * 4 * H, P.c = const_cast<float*>(c) + (long)t * B * H;  // (read)
    if (t > 0) P.c_prev = c + (long)(t - 1) * B * H;
    P.dh = (const float*)dh + (long)t * B * H;
    P.dG = (float*)w.big + (long)t * B * 4 * Hp, P.dc = w.dc_next;
    if (t + 1 < T_) P.dG_next = (const float*)w.big + (long)(t + 1) * B * 4 * Hp;
    P.B = B, P.H = H, P.Hk = Hk, P.Hp = Hp, P.off = a.ax.off, P.step = a.ax.step;
    ARD_LAUNCH(lstm_step32_bwd_kernel, dim3(ceil_div(Hp, 16), ceil_div(B, 16)), dim3(64 * kStepWaves), 0, stream, P);
    ARD_LAUNCH_CHECK("lstm_step32_bwd_kernel");
  }
  for (int t = one_launch || step32 ? -1 : T_ - 1; t >= 0; --t) {
    T* dGt = dG + (long)t * B * 4 * Hp;
    ARD_LAUNCH(lstm_cell_bwd_kernel<T>, cgrid, dim3(256), 0, stream, gates + (long)t * B * 4 * H,
                       c + (long)t * B * H, t > 0 ? c + (long)(t - 1) * B * H : (const float*)nullptr,
                       (const T*)dh + (long)t * B * H, dh_src, dh_splits, (long)B * Hp, w.dc_next, (const int*)w.rank, B, H,
                       Hk, Hp, t == T_ - 1 ? 1 : 0, dGt);
    ARD_LAUNCH_CHECK("lstm_cell_bwd_kernel");
    if (t > 0) {
      // dh_{t-1}[kept] = dG_t . Wh'
      GemmParams P = plain_gemm(dGt, 4 * Hp, w.whc, Hp, w.dh_next, Hp, B, Hp, 4 * Hp, true, false, ce, true, 0.0f);
      if (run_gemm_partials(a.dtype, true, false, P, stream, w.part, w.part_bytes, &dh_splits, &st)) {
        if (st) return st;
        dh_src = (const float*)w.part;
      } else {
        st = run_gemm(a.dtype, true, false, P, 0, 0, stream, w.part, w.part_bytes);
        if (st) return st;
        dh_src = w.dh_next;
        dh_splits = 1;
      }
    }
  }
  LstmScatter S{};
  void* dxo = Ip != I ? (void*)w.dxp : dx;
  {
    // dx[T*B x I] = dG . Wx', and the compact weight gradients dwx[4Hp x I] = dG^T . x, dwh[4Hp x Hp] = dG[1:]^T . h[kept][:-1]:
    // none needs another's result, so the bf16 ones of 64 x 64 tiles share a launch, each with partial sums of its own.
    // One after the other, each left CUs idle in its last round, or had fewer tiles than there are CUs (T = 64, B = 128,
    // I = H = 1024, dp = 2: 512 tiles, then 256, of 128 steps each).
    BatchOwn together;
    GemmParams Ph = plain_gemm(dG + (long)B * 4 * Hp, 4 * Hp, w.hc, Hp, w.dwh, Hp, 4 * Hp, Hp, (T_ - 1) * B, false, false, ce, false, 0.0f);
    GemmParams Px = plain_gemm(dG, 4 * Hp, xs, Ip, w.dwx, Ip, 4 * Hp, Ip, T_ * B, false, false, ce, false, 0.0f);
    if (lstm_sum_splits(a, Ip, Hp, w.part_bytes, Ph.sum_splits, Px.sum_splits)) {
      const size_t room_x = (size_t)Px.sum_splits * 16 * Hp * Ip;
      S.x = w.part, S.h = w.part + room_x;
      if (!run_gemm_partials(a.dtype, false, false, Px, stream, w.part, room_x, &S.nx, &st)) S.nx = 0;
      else if (!st && !run_gemm_partials(a.dtype, false, false, Ph, stream, w.part + room_x, w.part_bytes - room_x, &S.nh, &st)) S.nx = 0;
      if (st) return st;
    }
    if (!S.nx) {
      st = T_ > 1 ? run_gemm(a.dtype, false, false, Ph, 0, 0, stream, w.part, w.part_bytes) : fill_matrix(a.dtype, w.dwh, (long)4 * Hp * Hp, 0.0f, stream);
      if (st) return st;
      st = run_gemm(a.dtype, false, false, Px, 0, 0, stream, w.part_dwx, w.part_dwx_bytes);
      if (st) return st;
    }
    // (bf16 rows of whole words leave without their padding)
    if (Ip != I && a.es == 2 && I % 2 == 0 && ((uintptr_t)dx & 3) == 0 && !dev_knobs().no_fast && 4L * Hp * (T_ * (long)B > Ip ? T_ * (long)B : Ip) < (1L << 31) && (long)T_ * B * Ip < (1L << 31)) dxo = dx;
    GemmParams P = plain_gemm(dG, 4 * Hp, w.wxc, Ip, dxo, dxo == dx ? I : Ip, T_ * B, dxo == dx ? I : Ip, 4 * Hp, true, false, ce, false, 0.0f);
    if (a.es == 2) P.B.rpad = 1, P.B.vec = 1;  // (16-byte runs of the weights end in their padding)
    st = run_gemm(a.dtype, true, false, P, 0, 0, stream, w.part_dx, w.part_dx_bytes);
    if (st) return st;
    st = together.launch(stream);
    if (st) return st;
  }
  if (dxo != dx) {
    const long rows_total = (long)T_ * B;
    for (long r0 = 0; r0 < rows_total; r0 += 65535) {
      const long rows = rows_total - r0 < 65535 ? rows_total - r0 : 65535;
      ARD_LAUNCH(lstm_copy_rows_kernel<T>, dim3(ceil_div(I, 256), (unsigned)rows), dim3(256), 0, stream,
                         (const T*)w.dxp + r0 * Ip, (long)Ip, I, (long)I, (T*)dx + r0 * I);
      ARD_LAUNCH_CHECK("lstm_copy_rows_kernel");
    }
  }
  const int chunks = (I + H + 7) / 8, step = lstm_rows_per_launch(chunks);
  if (!S.nx) S.x = w.dwx, S.h = w.dwh;
  S.ax = a.ax, S.H = H, S.I = I, S.Ip = Ip, S.Hp = Hp, S.tp = a.tiles, S.dW = dW, S.rank = w.rank;
  S.by_chunks = fast_div((uint32_t)chunks), S.by_h = fast_div((uint32_t)H), S.by_step = fast_div((uint32_t)imax(a.ax.step, 1));
  for (S.p0 = 0; S.p0 < 4 * H; S.p0 = S.p1) {
    S.p1 = 4 * H - S.p0 < step ? 4 * H : S.p0 + step;
    const dim3 grid((unsigned)(((long)(S.p1 - S.p0) * chunks + 255) / 256));
    if constexpr (std::is_same<T, uint16_t>::value) {
      if (S.nx) {
        ARD_LAUNCH_NAMED(launch_instance("lstm_scatter_dw_kernel", S.nx, S.nh, 0), (lstm_scatter_dw_kernel<T, true, false>), grid, dim3(256), 0, stream, S);
        ARD_LAUNCH_CHECK("lstm_scatter_dw_kernel");
        continue;
      }
    }
    if (a.ax.kind == AX_AFFINE) ARD_LAUNCH_NAMED("lstm_scatter_dw_kernel", (lstm_scatter_dw_kernel<T, false, false>), grid, dim3(256), 0, stream, S);
    else ARD_LAUNCH_NAMED("lstm_scatter_dw_kernel", (lstm_scatter_dw_kernel<T, false, true>), grid, dim3(256), 0, stream, S);
    ARD_LAUNCH_CHECK("lstm_scatter_dw_kernel");
  }
  return ARD_OK;
}

}  // namespace ard

using namespace ard;

extern "C" size_t ard_lstm_workspace_bytes(int32_t dtype, int32_t T, int32_t B, int32_t I, int32_t H,
                                           const ard_pattern* pat) {
  LstmArgs a{dtype, T, B, I, H, 0, 0, Axis{}, LstmTiles{}};
  if (lstm_check(a, pat)) return 0;
  return lstm_ws_layout(nullptr, a.es, T, B, I, H, a.Hk).total;
}

extern "C" size_t ard_lstm_status_offset(int32_t dtype, int32_t T, int32_t B, int32_t I, int32_t H, const ard_pattern* pat) {
  LstmArgs a{dtype, T, B, I, H, 0, 0, Axis{}, LstmTiles{}};
  PersistPlan pp;
  if (lstm_check(a, pat) || (!lstm_xcd_fwd_units(a) && !lstm_staged_fwd_units(a) && !lstm_persist_plan(a, pp))) return (size_t)-1;
  const LstmWs w = lstm_ws_layout((char*)nullptr + 256, a.es, T, B, I, H, a.Hk);
  return (size_t)((char*)w.sync - ((char*)nullptr + 256));
}

extern "C" int32_t ard_lstm_fwd(int32_t dtype, int32_t T, int32_t B, int32_t I, int32_t H, const void* x,
                                const void* W, const ard_pattern* pat, void* h, float* c, float* gates, void* ws,
                                size_t ws_bytes, void* stream) {
  BatchSuspend not_recorded;  // this entry point's kernels depend on each other: never part of a grouped launch
  LstmArgs a{dtype, T, B, I, H, 0, 0, Axis{}, LstmTiles{}};
  int32_t st = lstm_check(a, pat);
  if (st) return st;
  if (!x || !W || !h || !c || !gates) return fail(ARD_EINVAL, "null tensor pointer");
  LstmWs w = lstm_ws_layout((char*)ws, a.es, T, B, I, H, a.Hk);
  if (!ws || ws_bytes < w.total) return fail(ARD_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", w.total, ws_bytes);
  if (dtype == ARD_BF16) return lstm_fwd_t<uint16_t>(a, x, W, h, c, gates, w, (hipStream_t)stream);
  return lstm_fwd_t<float>(a, x, W, h, c, gates, w, (hipStream_t)stream);
}

extern "C" int32_t ard_lstm_bwd(int32_t dtype, int32_t T, int32_t B, int32_t I, int32_t H, const void* x,
                                const void* W, const ard_pattern* pat, const void* h, const float* c,
                                const float* gates, const void* dh, void* dx, void* dW, void* ws, size_t ws_bytes,
                                void* stream) {
  BatchSuspend not_recorded;  // this entry point's kernels depend on each other: never part of a grouped launch
  LstmArgs a{dtype, T, B, I, H, 0, 0, Axis{}, LstmTiles{}};
  int32_t st = lstm_check(a, pat);
  if (st) return st;
  if (!x || !W || !h || !c || !gates || !dh || !dx || !dW) return fail(ARD_EINVAL, "null tensor pointer");
  LstmWs w = lstm_ws_layout((char*)ws, a.es, T, B, I, H, a.Hk);
  if (!ws || ws_bytes < w.total) return fail(ARD_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", w.total, ws_bytes);
  if (dtype == ARD_BF16) return lstm_bwd_t<uint16_t>(a, x, W, h, c, gates, dh, dx, dW, w, (hipStream_t)stream);
  return lstm_bwd_t<float>(a, x, W, h, c, gates, dh, dx, dW, w, (hipStream_t)stream);
}
