// One-mesh launches of the block form of the FP32 linear V-cycle (lin_block.h).
#include "lin_block.h"
#include "lin_block_launch.h"

namespace mr {

template <int TI, int TJ, int TK, int NT, bool ZERO>
__global__ void __launch_bounds__(NT) lin_down_kernel(LinDownArgs a) {
  __shared__ LinBoxLds<TI, TJ, TK, ZERO ? 4 : 5> sh;
  lin_down_body<TI, TJ, TK, NT, ZERO>(a, xcd_remap(blockIdx.x, gridDim.x), blockIdx.x, sh);
}

template <int TI, int TJ, int TK, int NT>
__global__ void __launch_bounds__(NT) lin_up_kernel(LinUpArgs a) {
  __shared__ LinBoxLds<TI, TJ, TK, 4> sh;
  lin_up_body<TI, TJ, TK, NT>(a, xcd_remap(blockIdx.x, gridDim.x), blockIdx.x, sh);
}

template <int NA, int NB, int NT>
__global__ void __launch_bounds__(NT) lin_tail2_kernel(LinTail2Args a) {
  __shared__ LinTail2Lds<NA, NB> sh;
  lin_tail2_body<NA, NB, NT>(a, sh);
}

hipError_t launch_lin_down(const LinDownArgs& a, hipStream_t s) {
  const LinBlkTile t = lin_blk_tile(a.n);
#define MR_LB_GO(TI, TJ, TK, NT)                                                                                     \
  if (t.ti == TI && t.tj == TJ && t.tk == TK) {                                                                      \
    if (a.e)                                                                                                         \
      hipLaunchKernelGGL((lin_down_kernel<TI, TJ, TK, NT, false>), dim3(lin_blk_blocks(a.n)), dim3(NT), 0, s, a);    \
    else                                                                                                             \
      hipLaunchKernelGGL((lin_down_kernel<TI, TJ, TK, NT, true>), dim3(lin_blk_blocks(a.n)), dim3(NT), 0, s, a);     \
    return hipGetLastError();                                                                                        \
  }
  MR_LB_TILES(MR_LB_GO)
#undef MR_LB_GO
  return hipErrorInvalidValue;
}

hipError_t launch_lin_up(const LinUpArgs& a, hipStream_t s) {
  const LinBlkTile t = lin_blk_tile(a.n);
#define MR_LB_GO(TI, TJ, TK, NT)                                                                          \
  if (t.ti == TI && t.tj == TJ && t.tk == TK) {                                                           \
    hipLaunchKernelGGL((lin_up_kernel<TI, TJ, TK, NT>), dim3(lin_blk_blocks(a.n)), dim3(NT), 0, s, a);    \
    return hipGetLastError();                                                                             \
  }
  MR_LB_TILES(MR_LB_GO)
#undef MR_LB_GO
  return hipErrorInvalidValue;
}

hipError_t launch_lin_tail2(const LinTail2Args& a, hipStream_t s) {
  if (a.n == 8)
    hipLaunchKernelGGL((lin_tail2_kernel<8, 4, 256>), dim3(1), dim3(256), 0, s, a);
  else if (a.n == 12)
    hipLaunchKernelGGL((lin_tail2_kernel<12, 6, 896>), dim3(1), dim3(896), 0, s, a);
  else if (a.n == 10)
    hipLaunchKernelGGL((lin_tail2_kernel<10, 0, 512>), dim3(1), dim3(512), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mr
