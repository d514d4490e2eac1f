// Launchers of the persistent FP32 tile kernels (batches of beams).
#include "win_dev.h"

namespace dd {

__global__ void zero_counter_kernel(int* c) {
  if (threadIdx.x < kNumXcd) c[threadIdx.x * kCounterStride] = 0;
}

hipError_t launch_batched(const Variant& v, const BeamDesc* d_beams, bool weighted, const int32_t* d_order,
                          const int32_t* d_qoff, int* d_counter, int grid, hipStream_t s) {
  const dim3 block(64 * v.nwave);
#define LAUNCH_P(ID, TP, DPW, NW, NWIN, CC, RC, NB, JMP)                                                    \
  if (v.id == ID) {                                                                                          \
    if (weighted)                                                                                            \
      hipLaunchKernelGGL((win_persistent<TP, DPW, NW, NWIN, CC, RC, NB, true, JMP>), dim3(grid), block, 0, s,  \
                         d_beams, d_order, d_qoff, d_counter);                                               \
    else                                                                                                     \
      hipLaunchKernelGGL((win_persistent<TP, DPW, NW, NWIN, CC, RC, NB, false, JMP>), dim3(grid), block, 0, s, \
                         d_beams, d_order, d_qoff, d_counter);                                               \
    return hipGetLastError();                                                                                \
  }
  if (v.kind == KIND_WIN_F32) {
    F32_VARIANTS(LAUNCH_P)
  }
#undef LAUNCH_P
  return hipErrorInvalidDeviceFunction;
}

int batched_blocks_per_cu(const Variant& v) {
  int n = 0;
#define OCC_P(ID, TP, DPW, NW, NWIN, CC, RC, NB, JMP)                                                            \
  if (v.id == ID) {                                                                                              \
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, win_persistent<TP, DPW, NW, NWIN, CC, RC, NB, false, JMP>, \
                                                     64 * NW, 0) != hipSuccess)                                   \
      n = 1;                                                                                                     \
    return n > 0 ? n : 1;                                                                                        \
  }
  if (v.kind == KIND_WIN_F32) {
    F32_VARIANTS(OCC_P)
  }
#undef OCC_P
  return 1;
}

hipError_t launch_zero_counter(int* d_counter, hipStream_t s) {
  hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(64), 0, s, d_counter);
  return hipGetLastError();
}

}  // namespace dd
