// Launcher of the FP32 tile kernels with the single-pulse search in their
// epilogue.
#include "win_dev.h"

namespace dd {

hipError_t launch_detect(const Variant& v, const TileArgs& a, int nbeam, hipStream_t s) {
  if (!detect_fusable(v)) return hipErrorInvalidDeviceFunction;
  const int64_t nblk = (int64_t)a.n_time_tiles * a.n_row_tiles;
  if (nblk < 1 || nblk > 0x7fffffff || nbeam < 1 || nbeam > 65535) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)nblk, (unsigned)nbeam);
  const dim3 block(64 * v.nwave);
  if (v.kind == KIND_WIN_F32) {
#define LAUNCH_DF(ID, TP, DPW, NW, NWIN, CC, RC, NB, JMP)                                                   \
  if constexpr (ID >= 13 && NB == 2) {                                                                        \
    if (v.id == ID) {                                                                                         \
      if (a.w_in)                                                                                             \
        hipLaunchKernelGGL((win_kernel<TP, DPW, NW, NWIN, CC, RC, NB, true, false, true, JMP>), grid, block, 0, \
                           s, a);                                                                             \
      else                                                                                                    \
        hipLaunchKernelGGL((win_kernel<TP, DPW, NW, NWIN, CC, RC, NB, false, false, true, JMP>), grid, block,   \
                           0, s, a);                                                                          \
      return hipGetLastError();                                                                               \
    }                                                                                                         \
  }
    F32_VARIANTS(LAUNCH_DF)
#undef LAUNCH_DF
  } else {
    return launch_detect_u8(v, a, grid, s);
  }
  return hipErrorInvalidDeviceFunction;
}

}  // namespace dd
