// Launchers of the FP32 tile kernels (win_dev.h) for the forward map and the
// adjoint, and the direct kernels.
#include <algorithm>

#include "win_dev.h"

namespace dd {

// ---------------------------------------------------------------------------
// Direct kernels: one work item per (output row, sample), one-dimensional
// blocks along time, every term read straight from global memory.  This is
// the paper's "generically tuned" form (Section 5: no DM-direction reuse) and
// the fallback for plans whose delay spans fit no tiled variant.
// ---------------------------------------------------------------------------
template <bool WEIGHTED>
__global__ __launch_bounds__(256) void direct_f32_kernel(const float* __restrict__ in, int64_t in_stride,
                                                         int64_t in_beam_stride, const int32_t* __restrict__ delta,
                                                         int nchan, const float* __restrict__ w, float* out,
                                                         int64_t out_stride, int64_t out_beam_stride, int nsamp,
                                                         int ntb) {
  const int j = blockIdx.x / ntb;
  const int t = (blockIdx.x - j * ntb) * 256 + threadIdx.x;
  const int b = blockIdx.y;
  if (t >= nsamp) return;
  const int32_t* drow = delta + (size_t)j * nchan;
  const float* src = in + (int64_t)b * in_beam_stride + t;
  float acc = 0.f;
  for (int c = 0; c < nchan; ++c) {
    const float x = src[(int64_t)c * in_stride + drow[c]];
    const float term = WEIGHTED ? w[c] * x : x;  // the weighted sample, rounded
    acc = acc + term;
  }
  out[(int64_t)b * out_beam_stride + (int64_t)j * out_stride + t] = acc;
}

__global__ __launch_bounds__(256) void direct_u8_kernel(const uint8_t* __restrict__ in, int64_t in_stride,
                                                        int64_t in_beam_stride, const int32_t* __restrict__ delta,
                                                        int nchan, int32_t* out, int64_t out_stride,
                                                        int64_t out_beam_stride, int nsamp, int ntb) {
  const int j = blockIdx.x / ntb;
  const int t = (blockIdx.x - j * ntb) * 256 + threadIdx.x;
  const int b = blockIdx.y;
  if (t >= nsamp) return;
  const int32_t* drow = delta + (size_t)j * nchan;
  const uint8_t* src = in + (int64_t)b * in_beam_stride + t;
  int32_t acc = 0;
  for (int c = 0; c < nchan; ++c) acc += (int32_t)src[(int64_t)c * in_stride + drow[c]];
  out[(int64_t)b * out_beam_stride + (int64_t)j * out_stride + t] = acc;
}

// Direct adjoint: one work item per (channel, input sample), summing over
// DM trials in ascending order; block partial sums of x * G for grad_w.
__global__ __launch_bounds__(256) void direct_adjoint_kernel(const float* __restrict__ g, int64_t g_stride,
                                                             int64_t g_beam_stride, const int32_t* __restrict__ delta,
                                                             int nchan, int ndm, int nsamp, int nin,
                                                             const float* __restrict__ w, float* grad_in,
                                                             int64_t gi_stride, int64_t gi_beam_stride,
                                                             const float* __restrict__ x, int64_t x_stride,
                                                             int64_t x_beam_stride, double* partial, int ntb) {
  __shared__ double red[256];
  const int c = blockIdx.x / ntb;
  const int tb = blockIdx.x - c * ntb;
  const int t = tb * 256 + threadIdx.x;
  const int b = blockIdx.y;
  float acc = 0.f;
  if (t < nin) {
    const float* gb = g + (int64_t)b * g_beam_stride;
    for (int j = 0; j < ndm; ++j) {
      const int s = t - delta[(size_t)j * nchan + c];
      if (s >= 0 && s < nsamp) acc = acc + gb[(int64_t)j * g_stride + s];
    }
    if (grad_in) grad_in[(int64_t)b * gi_beam_stride + (int64_t)c * gi_stride + t] = (w ? w[c] : 1.f) * acc;
  }
  if (partial) {
    double p = 0.0;
    if (t < nin) p = (double)x[(int64_t)b * x_beam_stride + (int64_t)c * x_stride + t] * (double)acc;
    red[threadIdx.x] = p;
    __syncthreads();
    for (int m = 128; m >= 1; m >>= 1) {
      if ((int)threadIdx.x < m) red[threadIdx.x] += red[threadIdx.x + m];
      __syncthreads();
    }
    if (threadIdx.x == 0) partial[((size_t)b * ntb + tb) * nchan + c] = red[0];
  }
}

// grad_w[c] = sum over parts p of partial[p][c], in FP64 and in a fixed order:
// thread row y of a block sums parts y, y + 32, ... of 32 channels, then the 32
// rows' sums are added in order: a short chain of loads whatever the number of
// parts (beams x time tiles).
constexpr int kGradwRows = 32, kGradwChans = 32;
__global__ __launch_bounds__(kGradwRows* kGradwChans) void reduce_gradw_kernel(const double* __restrict__ partial,
                                                                               int nparts, int nchan, float* grad_w) {
  __shared__ double sums[kGradwRows][kGradwChans];
  const int x = threadIdx.x % kGradwChans, y = threadIdx.x / kGradwChans;
  const int c = blockIdx.x * kGradwChans + x;
  double s = 0.0;
  if (c < nchan)
    for (int p = y; p < nparts; p += kGradwRows) s += partial[(size_t)p * nchan + c];
  sums[y][x] = s;
  __syncthreads();
  if (y != 0 || c >= nchan) return;
  for (int k = 1; k < kGradwRows; ++k) s += sums[k][x];
  grad_w[c] = (float)s;
}

const std::vector<Variant>& variants_f32() {
  static const std::vector<Variant> v = [] {
    std::vector<Variant> r;
#define MAKE_F32(ID, TP, DPW, NW, NWIN, CC, RC, NB, JMP)                                                    \
  r.push_back(Variant{JMP == 2 ? "win_tp" #TP "_dpw" #DPW "_nw" #NW "_win" #NWIN "_cc" #CC "_buf" #NB "_jmpf"   \
                      : JMP == 4 ? "win_tp" #TP "_dpw" #DPW "_nw" #NW "_win" #NWIN "_cc" #CC "_buf" #NB "_slots" \
                      : JMP    ? "win_tp" #TP "_dpw" #DPW "_nw" #NW "_win" #NWIN "_cc" #CC "_buf" #NB "_jmp"    \
                               : "win_tp" #TP "_dpw" #DPW "_nw" #NW "_win" #NWIN "_cc" #CC "_buf" #NB,         \
                      KIND_WIN_F32, TP, DPW, NW, NWIN, CC, RC, NB, ID, 0, JMP});
    F32_VARIANTS(MAKE_F32)
#undef MAKE_F32
    lane_variants(r);
    std::sort(r.begin(), r.end(), [](const Variant& a, const Variant& b) { return a.id < b.id; });
    return r;
  }();
  return v;
}

hipError_t launch_tiled(const Variant& v, const TileArgs& a, int nbeam, bool adjoint, hipStream_t s) {
  // uint8 double-buffered blocks walk tiles_per_block time tiles each
  const int tpb = (v.kind == KIND_TILE_U8 && v.nbuf == 2) ? a.tiles_per_block : 1;
  if (tpb < 1) return hipErrorInvalidConfiguration;
  const int64_t nblk = (int64_t)((a.n_time_tiles + tpb - 1) / tpb) * a.n_row_tiles;
  if (nblk < 1 || nblk > 0x7fffffff || nbeam < 1 || nbeam > 65535) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)nblk, (unsigned)nbeam);
  const dim3 block(64 * v.nwave);
  const bool weighted = adjoint ? false : (a.w_in != nullptr);
  if (v.kind == KIND_WIN_F32) {
#define LAUNCH_F32(ID, TP, DPW, NW, NWIN, CC, RC, NB, JMP)                                                      \
  if (v.id == ID) {                                                                                             \
    if (adjoint)                                                                                                \
      hipLaunchKernelGGL((win_kernel<TP, DPW, NW, NWIN, CC, RC, NB, false, true, false, JMP>), grid, block, 0, s, \
                         a);                                                                                    \
    else if (weighted)                                                                                          \
      hipLaunchKernelGGL((win_kernel<TP, DPW, NW, NWIN, CC, RC, NB, true, false, false, JMP>), grid, block, 0, s, \
                         a);                                                                                    \
    else                                                                                                        \
      hipLaunchKernelGGL((win_kernel<TP, DPW, NW, NWIN, CC, RC, NB, false, false, false, JMP>), grid, block, 0,   \
                         s, a);                                                                                 \
    return hipGetLastError();                                                                                   \
  }
    F32_VARIANTS(LAUNCH_F32)
#undef LAUNCH_F32
  } else if (v.kind == KIND_LANE_F32) {
    return launch_lane(v, a, grid, adjoint, s);
  } else {
    return launch_tiled_u8(v, a, grid, s);
  }
  return hipErrorInvalidDeviceFunction;
}

// Variants with the single-pulse search in their epilogue: the FP32 window
// variants from 13 on (asynchronous staging, the fastest ones) and every
// byte-shifted uint8 variant.
bool detect_fusable(const Variant& v) {
  return v.kind == KIND_WIN_F32 ? (v.id >= 13 && v.nbuf == 2) : v.kind == KIND_TILE_U8 && v.mode >= 1;
}

int det_step(const Variant& v) {
  const int run = v.kind == KIND_WIN_F32 ? v.tp : 4 * v.tp;  // window starts per lane
  return v.st() - run * ((kDetLook - 1 + run - 1) / run);
}

// 32-bit integer hash (a murmur3-style finaliser) of the word index.
__device__ __forceinline__ uint32_t hash32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

__global__ void fill_random_kernel(uint32_t* p, size_t nwords, bool f32, uint32_t seed) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nwords; i += (size_t)gridDim.x * blockDim.x) {
    const uint32_t h = hash32((uint32_t)i * 2654435761u + seed);
    p[i] = f32 ? __float_as_uint((float)(h >> 8) * (1.f / 8388608.f) - 1.f) : h;
  }
}

hipError_t launch_fill_random(void* p, size_t nbytes, bool f32, uint32_t seed, hipStream_t s) {
  const size_t nwords = nbytes / 4;  // a tail of < 4 bytes keeps its contents
  if (nwords == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((nwords + 255) / 256, 65536);
  hipLaunchKernelGGL(fill_random_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t*)p, nwords, f32, seed);
  return hipGetLastError();
}

hipError_t launch_direct_f32(const float* in, int64_t in_stride, int64_t in_beam_stride, const int32_t* delta,
                             int nchan, int ndm, const float* w, float* out, int64_t out_stride,
                             int64_t out_beam_stride, int nsamp, int nbeam, hipStream_t s) {
  const int ntb = (nsamp + 255) / 256;
  const int64_t gx = (int64_t)ntb * ndm;
  if (gx > 0x7fffffff || nbeam > 65535) return hipErrorInvalidConfiguration;
  if (w)
    hipLaunchKernelGGL(direct_f32_kernel<true>, dim3((unsigned)gx, nbeam), dim3(256), 0, s, in, in_stride,
                       in_beam_stride, delta, nchan, w, out, out_stride, out_beam_stride, nsamp, ntb);
  else
    hipLaunchKernelGGL(direct_f32_kernel<false>, dim3((unsigned)gx, nbeam), dim3(256), 0, s, in, in_stride,
                       in_beam_stride, delta, nchan, w, out, out_stride, out_beam_stride, nsamp, ntb);
  return hipGetLastError();
}

hipError_t launch_direct_u8(const uint8_t* in, int64_t in_stride, int64_t in_beam_stride, const int32_t* delta,
                            int nchan, int ndm, int32_t* out, int64_t out_stride, int64_t out_beam_stride,
                            int nsamp, int nbeam, hipStream_t s) {
  const int ntb = (nsamp + 255) / 256;
  const int64_t gx = (int64_t)ntb * ndm;
  if (gx > 0x7fffffff || nbeam > 65535) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(direct_u8_kernel, dim3((unsigned)gx, nbeam), dim3(256), 0, s, in, in_stride, in_beam_stride,
                     delta, nchan, out, out_stride, out_beam_stride, nsamp, ntb);
  return hipGetLastError();
}

hipError_t launch_direct_adjoint(const float* g, int64_t g_stride, int64_t g_beam_stride, const int32_t* delta,
                                 int nchan, int ndm, int nsamp, int nin, const float* w, float* grad_in,
                                 int64_t gi_stride, int64_t gi_beam_stride, const float* x, int64_t x_stride,
                                 int64_t x_beam_stride, double* partial, int nbeam, hipStream_t s) {
  const int ntb = (nin + 255) / 256;
  const int64_t gx = (int64_t)ntb * nchan;
  if (gx > 0x7fffffff || nbeam > 65535) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(direct_adjoint_kernel, dim3((unsigned)gx, nbeam), dim3(256), 0, s, g, g_stride, g_beam_stride,
                     delta, nchan, ndm, nsamp, nin, w, grad_in, gi_stride, gi_beam_stride, x, x_stride, x_beam_stride,
                     partial, ntb);
  return hipGetLastError();
}

hipError_t launch_reduce_gradw(const double* partial, int nparts, int nchan, float* grad_w, hipStream_t s) {
  hipLaunchKernelGGL(reduce_gradw_kernel, dim3((nchan + kGradwChans - 1) / kGradwChans), dim3(kGradwRows * kGradwChans), 0,
                     s, partial, nparts, nchan, grad_w);
  return hipGetLastError();
}

}  // namespace dd
