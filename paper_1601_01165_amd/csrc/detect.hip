// gfx950 kernels of the single-pulse search that do not dedisperse: the
// search over stored rows (the unfused path) and the merge of the per-tile
// records into one result per series.  The definition of the search and the
// tile records are in detect_dev.h.
#include <math.h>

#include <algorithm>

#include "detect_dev.h"
#include "internal.h"

namespace dd {

// The search over stored rows.  A tile's samples are the lanes' runs of
// kDetRowsRun; boxcar sums double, B_2w(i) = B_w(i) + B_w(i + w), and the sums past
// a lane's run are the next lane's own (DPP), so a sample costs one add per
// width.  Only each width's largest sum is kept: where it is reached is looked
// up afterwards in the one group of tiles that holds it (find_first).  That leaves
// about 16 vector issue slots per sample, 6 of them the FP64 moments, against 45
// when every lane summed its own 32-sample look-ahead and tracked positions.
constexpr int kRun = kDetRowsRun;

// The lane's run of the tile starting at sample t0; -inf past the row's end.
template <bool I32>
__device__ __forceinline__ void load_run(const void* rows, int64_t row_off, int t0, int nsamp, float* v) {
  const int pos = t0 + kRun * (threadIdx.x & 63);
  const int avail = nsamp - pos;
  if (I32) {
    const int32_t* src = static_cast<const int32_t*>(rows) + row_off + pos;
    if (avail >= kRun) {
#pragma unroll
      for (int i4 = 0; i4 < kRun / 4; ++i4) {
        const int4 x = reinterpret_cast<const int4*>(src)[i4];
        v[4 * i4 + 0] = (float)x.x;
        v[4 * i4 + 1] = (float)x.y;
        v[4 * i4 + 2] = (float)x.z;
        v[4 * i4 + 3] = (float)x.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kRun; ++i) v[i] = i < avail ? (float)src[i] : -INFINITY;
    }
  } else {
    const float* src = static_cast<const float*>(rows) + row_off + pos;
    if (avail >= kRun) {
#pragma unroll
      for (int i4 = 0; i4 < kRun / 4; ++i4) {
        const float4 x = reinterpret_cast<const float4*>(src)[i4];
        v[4 * i4 + 0] = x.x;
        v[4 * i4 + 1] = x.y;
        v[4 * i4 + 2] = x.z;
        v[4 * i4 + 3] = x.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kRun; ++i) v[i] = i < avail ? src[i] : -INFINITY;
    }
  }
}

// Boxcar sums of width w to width 2 w, in place.  The last lane's sums past
// its run become -inf (its starts belong to the next tile).
template <int W>
__device__ __forceinline__ void double_width(float* v) {
  static_assert(W <= kRun, "the sums past a run are the next lane's");
  float next[W];
#pragma unroll
  for (int j = 0; j < W; ++j)
    next[j] = __int_as_float(det_next_lane(__float_as_int(-INFINITY), __float_as_int(v[j])));
#pragma unroll
  for (int i = 0; i < kRun; ++i) v[i] = v[i] + (i + W < kRun ? v[i + W < kRun ? i + W : 0] : next[i + W < kRun ? 0 : i + W - kRun]);
}

template <int K>
__device__ __forceinline__ void run_max(float* v, float* best) {
  if constexpr (K > 0) double_width<1 << (K - 1)>(v);
  float m = best[K];
#pragma unroll
  for (int i = 0; i < kRun; i += 2) m = fmaxf(fmaxf(m, v[i]), v[i + 1]);
  best[K] = m;
  if constexpr (K + 1 < kDetNW) run_max<K + 1>(v, best);
}

// Tiles [ta, tb) of a row by one wave: each width's largest sum and the moments
// (of the whole wave, in every lane).
template <bool I32>
__device__ __forceinline__ void wave_tiles(const void* rows, int64_t row_off, int nsamp, int ta, int tb, float* m,
                                           double& s1, double& s2) {
  const int lane = threadIdx.x & 63;
  const bool owned = kRun * lane < kDetRowsStep;
  float best[kDetNW];
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) best[k] = -INFINITY;
  s1 = 0.0;
  s2 = 0.0;
  float v[kRun], nv[kRun];
  load_run<I32>(rows, row_off, ta * kDetRowsStep, nsamp, nv);
  for (int tt = ta; tt < tb; ++tt) {
    const int t0 = tt * kDetRowsStep;
#pragma unroll
    for (int i = 0; i < kRun; ++i) v[i] = nv[i];
    if (tt + 1 < tb) load_run<I32>(rows, row_off, t0 + kDetRowsStep, nsamp, nv);
    if (owned) {
      const int lim = nsamp - t0 - kRun * lane;  // the lane's starts that hold samples
      if (lim >= kRun) {
#pragma unroll
        for (int i = 0; i < kRun; ++i) {
          const double y = (double)v[i];
          s1 += y;
          s2 = fma(y, y, s2);
        }
      } else {
#pragma unroll
        for (int i = 0; i < kRun; ++i)
          if (i < lim) {
            const double y = (double)v[i];
            s1 += y;
            s2 = fma(y, y, s2);
          }
      }
    }
    run_max<0>(v, best);
  }
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) m[k] = det_wave_maxf(owned ? best[k] : -INFINITY);
  s1 = det_wave_sum(s1);
  s2 = det_wave_sum(s2);
}

// One wave per row and group of `group` consecutive tiles.
template <bool I32>
__global__ __launch_bounds__(256) void detect_rows_kernel(const void* __restrict__ rows, int64_t stride, int nrows,
                                                          int nsamp, int ntiles, int group, int ngroups,
                                                          DetRec* __restrict__ recs) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = blockIdx.x % ngroups;
  const int r = (blockIdx.x / ngroups) * 4 + wave;
  if (r >= nrows) return;  // whole waves; no block barrier follows
  float m[kDetNW];
  double s1, s2;
  wave_tiles<I32>(rows, (int64_t)r * stride, nsamp, g * group, min(ntiles, (g + 1) * group), m, s1, s2);
  if (lane == 0) {
    int4* o = reinterpret_cast<int4*>(recs + (int64_t)r * ngroups + g);
    o[0] = make_int4(__float_as_int(m[0]), __float_as_int(m[1]), __float_as_int(m[2]), __float_as_int(m[3]));
    o[1] = make_int4(__float_as_int(m[4]), __float_as_int(m[5]), 0, 0);
    o[2] = make_int4(0, 0, 0, 0);
    double2 s;
    s.x = s1;
    s.y = s2;
    *reinterpret_cast<double2*>(o + 3) = s;
  }
}

// The first start in tiles [ta, tb) of a row whose boxcar of width 2^kw sums to m
// (the same additions as the search's, so the sum is found exactly).
template <bool I32>
__device__ int find_first(const void* rows, int64_t row_off, int nsamp, int ta, int tb, int kw, float m) {
  const int lane = threadIdx.x & 63;
  for (int tt = ta; tt < tb; ++tt) {
    float v[kRun];
    load_run<I32>(rows, row_off, tt * kDetRowsStep, nsamp, v);
    if (kw > 0) double_width<1>(v);
    if (kw > 1) double_width<2>(v);
    if (kw > 2) double_width<4>(v);
    if (kw > 3) double_width<8>(v);
    if (kw > 4) double_width<16>(v);
    int at = -1;
#pragma unroll
    for (int i = kRun - 1; i >= 0; --i) at = v[i] == m ? i : at;
    const uint64_t hit = __ballot(at >= 0 && kRun * lane < kDetRowsStep);
    if (hit) {
      const int l0 = __builtin_ctzll(hit);
      return tt * kDetRowsStep + kRun * l0 + __builtin_amdgcn_readlane(at, l0);
    }
  }
  return -1;
}

// Mean, standard deviation and the best width of a series from its moments and
// each width's largest sum (valid[k]: some window of the width fits):
//   S/N_w = (max B_w - w mean) / (std sqrt(w)), 0 when std == 0.
// Returns the index of the best width, -1 if none fits.
__device__ __forceinline__ int det_score(double s1, double s2, int nsamp, int nwidth, const double* m, const bool* valid,
                                         double& best, double& mu, double& sd) {
  const double n = (double)nsamp;
  mu = s1 / n;
  double var = (s2 - s1 * mu) / n;
  if (!(var > 0.0)) var = 0.0;
  sd = sqrt(var);
  best = 0.0;
  int kb = -1;
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) {
    if (k >= nwidth || !valid[k]) continue;
    const double w = (double)(1 << k);
    const double sn = sd > 0.0 ? (m[k] - w * mu) / (sd * sqrt(w)) : 0.0;
    if (kb < 0 || sn > best) {
      best = sn;
      kb = k;
    }
  }
  return kb;
}

// One wave per stored row: merges the row's records, scores the widths and
// looks up where the best one's largest sum is first reached.
template <bool I32>
__global__ __launch_bounds__(256) void det_finish_rows_kernel(const DetRec* __restrict__ recs,
                                                              const void* __restrict__ rows, int64_t stride, int nrows,
                                                              int ntiles, int group, int ngroups, int nsamp, int nwidth,
                                                              double* __restrict__ snr, int32_t* __restrict__ width,
                                                              int32_t* __restrict__ start, double* __restrict__ mean,
                                                              double* __restrict__ stdv) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + wave;
  if (r >= nrows) return;
  const DetRec* R = recs + (int64_t)r * ngroups;
  float bf[kDetNW];
  int bg[kDetNW];
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) {
    bf[k] = -INFINITY;
    bg[k] = INT32_MAX;
  }
  double s1 = 0.0, s2 = 0.0;
  for (int g = lane; g < ngroups; g += 64) {
    const DetRec rec = R[g];
#pragma unroll
    for (int k = 0; k < kDetNW; ++k) {
      const float f = __int_as_float(rec.val[k]);
      if (f > bf[k]) {
        bf[k] = f;
        bg[k] = g;
      }
    }
    s1 += rec.s1;
    s2 += rec.s2;
  }
  s1 = det_wave_sum(s1);
  s2 = det_wave_sum(s2);
  double m[kDetNW];
  bool valid[kDetNW];
  int first[kDetNW];
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) {
    const float mm = det_wave_maxf(bf[k]);
    first[k] = det_wave_min(bf[k] == mm ? bg[k] : INT32_MAX);
    valid[k] = first[k] != INT32_MAX;
    m[k] = (double)mm;
  }
  double best, mu, sd;
  const int kb = __builtin_amdgcn_readfirstlane(det_score(s1, s2, nsamp, nwidth, m, valid, best, mu, sd));
  int at = -1;
  if (kb >= 0) {
    float top = (float)m[0];
    int g = first[0];
#pragma unroll
    for (int k = 1; k < kDetNW; ++k)
      if (k == kb) {
        top = (float)m[k];
        g = first[k];
      }
    at = find_first<I32>(rows, (int64_t)r * stride, nsamp, g * group, min(ntiles, (g + 1) * group), kb, top);
  }
  if (lane != 0) return;
  snr[r] = best;
  width[r] = kb < 0 ? -1 : 1 << kb;
  start[r] = at;
  if (mean) mean[r] = mu;
  if (stdv) stdv[r] = sd;
}

// The whole search of a row by one block, its waves taking consecutive shares of
// the tiles: no records, and no second launch whose few microseconds of latency
// (loading records, scoring, loading the tiles again) nothing hides.  Bound by the read of
// the rows: 2,000 rows of 20,000 samples in 33.7 us (4.7 TB/s) against 39.7 in two launches
// (28 + 9), 818 rows of 9,090 in 23.5 against 27.  launch_detect_rows says which rows
// take it.
template <bool I32, int NW>
__global__ __launch_bounds__(64 * NW) void search_row_kernel(const void* __restrict__ rows, int64_t stride, int nsamp,
                                                             int ntiles, int nwidth, double* __restrict__ snr,
                                                             int32_t* __restrict__ width, int32_t* __restrict__ start,
                                                             double* __restrict__ mean, double* __restrict__ stdv) {
  __shared__ float wm[NW][kDetNW];
  __shared__ double ws[NW][2];
  __shared__ int found[NW];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = blockIdx.x;
  const int64_t row_off = (int64_t)r * stride;
  const int share = (ntiles + NW - 1) / NW;
  float m[kDetNW];
  double s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) m[k] = -INFINITY;
  if (wave * share < ntiles)
    wave_tiles<I32>(rows, row_off, nsamp, wave * share, min(ntiles, (wave + 1) * share), m, s1, s2);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < kDetNW; ++k) wm[wave][k] = m[k];
    ws[wave][0] = s1;
    ws[wave][1] = s2;
  }
  __syncthreads();
  // every wave merges and scores, so that all know where to look
  s1 = ws[0][0];
  s2 = ws[0][1];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    s1 += ws[w][0];
    s2 += ws[w][1];
  }
  double md[kDetNW];
  bool valid[kDetNW];
  int first[kDetNW];
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) {
    float top = -INFINITY;
    first[k] = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = wm[w][k];
      first[k] = f > top ? w : first[k];
      top = f > top ? f : top;
    }
    valid[k] = top > -INFINITY;
    md[k] = (double)top;
  }
  double best, mu, sd;
  const int kb = __builtin_amdgcn_readfirstlane(det_score(s1, s2, nsamp, nwidth, md, valid, best, mu, sd));
  if (kb >= 0) {
    float top = (float)md[0];
    int w0 = first[0];
#pragma unroll
    for (int k = 1; k < kDetNW; ++k)
      if (k == kb) {
        top = (float)md[k];
        w0 = first[k];
      }
    w0 = __builtin_amdgcn_readfirstlane(w0);
    int at = -1;
    const int tb = min(ntiles, (w0 + 1) * share);
    for (int tt = w0 * share + wave; tt < tb && at < 0; tt += NW)
      at = find_first<I32>(rows, row_off, nsamp, tt, tt + 1, kb, top);
    if (lane == 0) found[wave] = at;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  int at = -1;
  if (kb >= 0)
    for (int w = 0; w < NW; ++w)
      if (found[w] >= 0 && (at < 0 || found[w] < at)) at = found[w];
  snr[r] = best;
  width[r] = kb < 0 ? -1 : 1 << kb;
  start[r] = at;
  if (mean) mean[r] = mu;
  if (stdv) stdv[r] = sd;
}

// One wave per series: lane k takes tiles k, k + 64, ... in order (keeping
// the first of equal sums), then the lanes merge (largest sum, then smallest
// start), the moments are summed in a fixed order, and lane 0 scores the
// widths (det_score).
template <bool INT_VALS>
__global__ __launch_bounds__(256) void det_finish_kernel(const DetRec* __restrict__ recs, int nseries, int ntiles,
                                                         int nsamp, int nwidth, double* __restrict__ snr,
                                                         int32_t* __restrict__ width, int32_t* __restrict__ start,
                                                         double* __restrict__ mean, double* __restrict__ stdv) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int sidx = blockIdx.x * 4 + wave;
  if (sidx >= nseries) return;
  const DetRec* R = recs + (int64_t)sidx * ntiles;
  float bf[kDetNW];
  int bi[kDetNW], bp[kDetNW];
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) {
    bf[k] = -INFINITY;
    bi[k] = INT32_MIN;
    bp[k] = -1;
  }
  double s1 = 0.0, s2 = 0.0;
  for (int t = lane; t < ntiles; t += 64) {
    const DetRec rec = R[t];
#pragma unroll
    for (int k = 0; k < kDetNW; ++k) {
      if (rec.pos[k] < 0) continue;
      if (INT_VALS) {
        if (bp[k] < 0 || rec.val[k] > bi[k]) {
          bi[k] = rec.val[k];
          bp[k] = rec.pos[k];
        }
      } else {
        const float f = __int_as_float(rec.val[k]);
        if (bp[k] < 0 || f > bf[k]) {
          bf[k] = f;
          bp[k] = rec.pos[k];
        }
      }
    }
    s1 += rec.s1;
    s2 += rec.s2;
  }
  s1 = det_wave_sum(s1);
  s2 = det_wave_sum(s2);
  double m[kDetNW];
  int p[kDetNW];
  bool valid[kDetNW];
#pragma unroll
  for (int k = 0; k < kDetNW; ++k) {
    if (INT_VALS) {
      const int mm = det_wave_max(bp[k] >= 0 ? bi[k] : INT32_MIN);
      p[k] = det_wave_min(bp[k] >= 0 && bi[k] == mm ? bp[k] : INT32_MAX);
      m[k] = (double)mm;
    } else {
      const float mm = det_wave_maxf(bp[k] >= 0 ? bf[k] : -INFINITY);
      p[k] = det_wave_min(bp[k] >= 0 && bf[k] == mm ? bp[k] : INT32_MAX);
      m[k] = (double)mm;
    }
    valid[k] = p[k] != INT32_MAX;  // some window of this width fits
  }
  if (lane != 0) return;
  double best, mu, sd;
  const int kb = det_score(s1, s2, nsamp, nwidth, m, valid, best, mu, sd);
  int bs = -1;
#pragma unroll
  for (int k = 0; k < kDetNW; ++k)
    if (k == kb) bs = p[k];
  snr[sidx] = best;
  width[sidx] = kb < 0 ? -1 : 1 << kb;
  start[sidx] = bs;
  if (mean) mean[sidx] = mu;
  if (stdv) stdv[sidx] = sd;
}

// Tiles one wave of the row search's first launch takes: enough waves to fill the
// chip about twice come first (300 rows of 100,000 samples: 30,300 tiles in groups of 3);
// longer groups then save wave reductions and records.
static int rows_group(int nrows, int ntiles) {
  const int64_t tiles = (int64_t)nrows * ntiles;
  return (int)std::max<int64_t>(1, std::min<int64_t>({tiles / 8192, ntiles, 8}));
}

// Work items of one launch (a 32-bit count).
static constexpr int64_t kMaxWorkItems = 0xffffffffll;

hipError_t launch_detect_rows(const void* rows, bool i32, int64_t stride, int nrows, int nsamp, int ntiles, int nwidth,
                              DetRec* recs, double* snr, int32_t* width, int32_t* start, double* mean, double* stdv,
                              hipStream_t s) {
  if (nrows < 1 || ntiles < 1) return hipErrorInvalidConfiguration;
  // A block of four waves per row while a wave's share of the tiles is short: up to 32
  // tiles, or 12 where there are fewer rows than would fill the chip (GPU times in us, one
  // launch against two: 255 rows of 32 tiles 10.5 and 12.3, of 12 tiles 6.6 and 8.5; 64 rows of
  // 32 tiles 9.9 and 7.8, of 12 tiles 6.5 and 7.4; 300 rows of 101 tiles 42 and 27).  One
  // wave where four would have no tile each: 100,000 rows of 500 samples 116 us, 314 with four waves; 6,000
  // rows of 3 tiles level; 50,000 rows of 2 tiles 102 and 180.  Few such rows of 2 or 3 tiles keep four
  // (64 rows of 3: 5.1 and 6.9).  One wave too where four a row would be 2^32 work items.
  if (ntiles <= (nrows < 192 ? 12 : 32)) {
    auto launch = [&](auto kernel, int nw) {
      if ((int64_t)nrows * 64 * nw > kMaxWorkItems) return hipErrorInvalidConfiguration;
      hipLaunchKernelGGL(kernel, dim3((unsigned)nrows), dim3(64 * nw), 0, s, rows, stride, nsamp, ntiles, nwidth, snr,
                         width, start, mean, stdv);
      return hipGetLastError();
    };
    const bool one = ntiles == 1 || (ntiles <= 3 && nrows >= 4096) || (int64_t)nrows * 256 > kMaxWorkItems;
    if (one) return i32 ? launch(search_row_kernel<true, 1>, 1) : launch(search_row_kernel<false, 1>, 1);
    return i32 ? launch(search_row_kernel<true, 4>, 4) : launch(search_row_kernel<false, 4>, 4);
  }
  const int group = rows_group(nrows, ntiles), ngroups = (ntiles + group - 1) / group;
  const int64_t nblk = (int64_t)ngroups * ((nrows + 3) / 4);
  if (nblk * 256 > kMaxWorkItems) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)nblk), fin((unsigned)((nrows + 3) / 4));
  if (i32) {
    hipLaunchKernelGGL((detect_rows_kernel<true>), grid, dim3(256), 0, s, rows, stride, nrows, nsamp, ntiles, group,
                       ngroups, recs);
    hipLaunchKernelGGL((det_finish_rows_kernel<true>), fin, dim3(256), 0, s, recs, rows, stride, nrows, ntiles, group,
                       ngroups, nsamp, nwidth, snr, width, start, mean, stdv);
  } else {
    hipLaunchKernelGGL((detect_rows_kernel<false>), grid, dim3(256), 0, s, rows, stride, nrows, nsamp, ntiles, group,
                       ngroups, recs);
    hipLaunchKernelGGL((det_finish_rows_kernel<false>), fin, dim3(256), 0, s, recs, rows, stride, nrows, ntiles, group,
                       ngroups, nsamp, nwidth, snr, width, start, mean, stdv);
  }
  return hipGetLastError();
}

hipError_t launch_det_finish(const DetRec* recs, bool int_vals, int nseries, int ntiles, int nsamp, int nwidth,
                             double* snr, int32_t* width, int32_t* start, double* mean, double* stdv, hipStream_t s) {
  if (nseries < 1 || ntiles < 1) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)((nseries + 3) / 4));
  if (int_vals)
    hipLaunchKernelGGL((det_finish_kernel<true>), grid, dim3(256), 0, s, recs, nseries, ntiles, nsamp, nwidth, snr,
                       width, start, mean, stdv);
  else
    hipLaunchKernelGGL((det_finish_kernel<false>), grid, dim3(256), 0, s, recs, nseries, ntiles, nsamp, nwidth, snr,
                       width, start, mean, stdv);
  return hipGetLastError();
}

}  // namespace dd
