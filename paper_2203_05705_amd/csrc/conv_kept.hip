// The kernels of conv_blocks.hpp and conv_scatter.hpp, in a file of their own: in one code object with
// those of conv.hip a small product's launch there took 1.1 us longer (16 x 38 channels of 32 x 32 -> 146, forward 10.4 -> 9.2 us).
#include "conv_blocks.hpp"
#include "conv_scatter.hpp"

namespace ard {

template <class P> static int32_t block_launch(void (*kernel)(P), const char* name, const P& p, hipStream_t stream, bool& raised) {
  if (!raised) {
    ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, kBlockLds));
    raised = !dry_run();
  }
  ARD_LAUNCH_NAMED(name, kernel, dim3((unsigned)(ceil_div(p.total, 8) * 8)), dim3(256), kBlockLds, stream, p);
  ARD_LAUNCH_CHECK(name);
  return ARD_OK;
}
int32_t launch_conv_block_fwd(const BlockFwdParams& P, hipStream_t stream) {
  static thread_local bool raised = false;
  return block_launch(conv_block_fwd_kernel, "conv_block_fwd_kernel", P, stream, raised);
}
int32_t launch_conv_block_data(const BlockDataParams& P, hipStream_t stream) {
  static thread_local bool raised = false;
  return block_launch(conv_block_data_kernel, "conv_block_data_kernel", P, stream, raised);
}

template <int KS> static int32_t scatter_launch(const ScatterDataParams& P, hipStream_t stream) {
  auto kernel = conv_scatter_data_kernel<KS>;
  static thread_local bool raised = false;
  if (!raised) {
    ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, kSdMostLds));
    raised = !dry_run();
  }
  ARD_LAUNCH_NAMED("conv_scatter_data_kernel", kernel, dim3((unsigned)(ceil_div(P.total, 8) * 8)), dim3(256), (size_t)P.lds_bytes, stream, P);
  ARD_LAUNCH_CHECK("conv_scatter_data_kernel");
  return ARD_OK;
}
int32_t launch_conv_scatter(int ks, const ScatterDataParams& P, hipStream_t stream) {
  return ks == 8 ? scatter_launch<8>(P, stream) : ks == 6 ? scatter_launch<6>(P, stream) : ks == 4 ? scatter_launch<4>(P, stream) : scatter_launch<2>(P, stream);
}

}  // namespace ard
