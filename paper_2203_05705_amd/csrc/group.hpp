// Kernel of the grouped launches.
#pragma once
#include "engine.hpp"
#include "fast.hpp"
#include "skinny.hpp"
#include "small.hpp"

namespace ard {

// Wc[r][c] = W[out(r)][in(c)]; rows and columns up to the next multiple of 8 are zero
struct CompactWArgs {
  const void* W;
  void* Wc;
  long ld;
  Axis ao, ai;
};
// a workgroup gathers kCwRows rows x 256 columns: a thread's loads of its rows are independent and in
// flight together
constexpr int kCwRows = 16;
template <typename T>
__device__ __forceinline__ void compact_weight_body(const CompactWArgs& a, const int bx, const int by) {
  const int c = bx * 256 + threadIdx.x;
  const int cols = pad8(a.ai.n), rows = pad8(a.ao.n);
  if (c >= cols) return;
  const T* W = reinterpret_cast<const T*>(a.W);
  T* Wc = reinterpret_cast<T*>(a.Wc);
  const bool c_ok = c < a.ai.n;
  const long pc = c_ok ? ax_phys(a.ai, c) : 0;
  T v[kCwRows];
#pragma unroll
  for (int i = 0; i < kCwRows; ++i) {
    const int r = by * kCwRows + i;
    const bool ok = c_ok && r < a.ao.n;
    const T t = W[(long)(ok ? ax_phys(a.ao, r) : 0) * a.ld + pc];  // unconditional (clamped) load
    v[i] = ok ? t : (T)0;
  }
#pragma unroll
  for (int i = 0; i < kCwRows; ++i) {
    const int r = by * kCwRows + i;
    if (r < rows) Wc[(long)r * cols + c] = v[i];
  }
}
}  // namespace ard

// ---- grouped launches ----------------------------------------------------------------------------
//
// A training iteration of a small layer chain is a handful of products of a few microseconds each,
// so what it costs is mostly the fixed part of every launch.  Calls that do not depend on each other
// (the weight compaction and the first forward product; the three products of the classifier layer;
// the weight and data gradients of a hidden layer) can be recorded and then issued as one grid of
// group_kernel, which holds the bodies of every kernel such a chain uses (all run 256 threads per
// workgroup); each workgroup looks up the segment of the grid it belongs to and runs that body.
namespace ard {

constexpr int kGroupMaxSeg = 6;
constexpr int kGroupArgBytes = 3584;
struct GroupSeg {
  int kind;      // GK_*
  int first;     // first workgroup of the segment (a multiple of 8: workgroup ids go round-robin over the XCDs)
  int nblocks;   // gx * gy
  int gx, gy;
  int arg_off;   // byte offset of the body's argument struct in GroupTable::args
};
struct GroupTable {
  int nseg;
  GroupSeg seg[kGroupMaxSeg];
  alignas(16) char args[kGroupArgBytes];
};
static_assert(sizeof(GroupTable) <= 4096, "kernel arguments are limited to 4 KiB");

// (The table is read through the kernel-argument segment itself: indexing the by-value parameter with a
// run-time segment number would make the compiler copy all of it into every lane's private memory.)
// SMALL: with the bodies of small.hpp, in a kernel and a file of its own: with them among its neighbours the others' launches
// took 0.2 us longer each (training step of 1024 x 784 -> 2048 -> 2048 -> 10 55.7 against 56.3 us).
template <bool SMALL>
__global__ __launch_bounds__(256, 2) void group_kernel(const GroupTable table_in_kernarg) {
  extern __shared__ uint4 group_lds[];
  const GroupTable& T = *(const GroupTable*)__builtin_amdgcn_kernarg_segment_ptr();
  int s = 0;
  while (s + 1 < T.nseg && (int)blockIdx.x >= T.seg[s + 1].first) ++s;
  const GroupSeg sg = T.seg[s];
  const int local = (int)blockIdx.x - sg.first;
  if (local >= sg.nblocks) return;
  const char* arg = T.args + sg.arg_off;
  switch (sg.kind) {
    case GK_DIRECT_KK_64:
      direct_body<true, true, 64, 64, 4, 0>(*reinterpret_cast<const FastParams*>(arg), local, group_lds);
      break;
    case GK_DIRECT_KM_64:
      direct_body<true, false, 64, 64, 4, 0>(*reinterpret_cast<const FastParams*>(arg), local, group_lds);
      break;
    case GK_DIRECT_MM_64:
      direct_body<false, false, 64, 64, 4, 0>(*reinterpret_cast<const FastParams*>(arg), local, group_lds);
      break;
    case GK_DIRECT_MM_128x64:
      direct_body<false, false, 128, 64, 4, 0>(*reinterpret_cast<const FastParams*>(arg), local, group_lds);
      break;
    case GK_SKINNY_FWD:
      skinny_fwd_body(*reinterpret_cast<const SkinnyArgs*>(arg), local, group_lds);
      break;
    case GK_SKINNY_BWD_DATA:
      skinny_bwd_data_body(*reinterpret_cast<const SkinnyArgs*>(arg), local % sg.gx, local / sg.gx, group_lds);
      break;
    case GK_SKINNY_BWD_WEIGHT:
      skinny_bwd_weight_body(*reinterpret_cast<const SkinnyArgs*>(arg), local, group_lds);
      break;
    case GK_COMPACT_W:
      compact_weight_body<uint16_t>(*reinterpret_cast<const CompactWArgs*>(arg), local % sg.gx, local / sg.gx);
      break;
    case GK_FINISH_VEC:
      finish_vec_body(*reinterpret_cast<const FinishArgs*>(arg), local % sg.gx, local / sg.gx, sg.gy);
      break;
    case GK_ZERO_ROWS:
      zero_rows_body(*reinterpret_cast<const ZeroRowsArgs*>(arg), local, sg.nblocks);
      break;
    default:
      if constexpr (SMALL) small_recorded(sg.kind, [&](auto v) {
          small_body<v.a_kc, v.b_kc, v.sa, v.sb, 2>(*reinterpret_cast<const SmallArgs*>(arg), local, 256, group_lds);
        });
      break;
  }
}

// (small.hip) the grouped launch with the bodies of small.hpp
int32_t launch_group_small(const GroupTable& T, int blocks, size_t lds, hipStream_t stream);
// the most LDS that a recorded kernel asks for
constexpr int kGroupMaxLds = 4096 + 16 * (SK_MAX_COLS + 16) * 2 + 256;

}  // namespace ard
