// The kernels of small.hpp and the grouped launch that holds their bodies beside the others.
#include <type_traits>

#include "group.hpp"

namespace ard {

template <bool A_KC, bool B_KC, int SA, int SB>
__global__ __launch_bounds__(512) void gemm_small_kernel(const SmallArgs P) {
  __shared__ uint4 lds[small_lds_bytes(8) / 16 + 1];
  small_body<A_KC, B_KC, SA, SB, 1>(P, (int)blockIdx.x, (int)blockDim.x, lds);
}

void launch_small_alone(int kind, const SmallArgs& P, unsigned tiles, unsigned threads, hipStream_t stream) {
  auto launch = [&](auto v) {
    using V = decltype(v);
    ARD_LAUNCH_NAMED("gemm_small_kernel", (gemm_small_kernel<V::a_kc, V::b_kc, V::sa, V::sb>), dim3(tiles), dim3(threads), 0, stream, P);
  };
  if (small_recorded(kind, launch)) return;
  switch (kind) {
    case GK_SMALL_KK + 2: return launch(SmallForm<true, true, 2, 2>{});
    case GK_SMALL_KK + 3: return launch(SmallForm<true, true, 3, 3>{});
    case GK_SMALL_KK + 4: return launch(SmallForm<true, true, 4, 4>{});
    case GK_SMALL_KM + 0: return launch(SmallForm<true, false, 0, 0>{});
    case GK_SMALL_KM + 2: return launch(SmallForm<true, false, 2, 0>{});
    case GK_SMALL_KM + 3: return launch(SmallForm<true, false, 3, 0>{});
    case GK_SMALL_KM + 4: return launch(SmallForm<true, false, 4, 0>{});
    default: return launch(SmallForm<true, true, 0, 0>{});
  }
}

int32_t launch_group_small(const GroupTable& T, int blocks, size_t lds, hipStream_t stream) {
  static thread_local bool raised = false;
  if (!raised) {
    ARD_HIP_CHECK(raise_lds_limit((const void*)group_kernel<true>, kGroupMaxLds));
    raised = !dry_run();
  }
  ARD_LAUNCH_NAMED("group_kernel", group_kernel<true>, dim3((unsigned)blocks), dim3(256), lds, stream, T);
  ARD_LAUNCH_CHECK("group_kernel");
  return ARD_OK;
}

}  // namespace ard
