// Tile tables built on the GPU from the plan's delay matrix (what they hold is
// described with struct Tables), those of several variants in one launch.
#include <algorithm>

#include "internal.h"

namespace dd {

namespace {

// Delay of output row r for input row c: the plan's matrix, or its transpose
// counted down from `pad` (adjoint).
struct DelayView {
  const int32_t* delta;
  int nchan;
  bool adj;
  int pad;
  __device__ int operator()(int r, int c) const {
    return adj ? pad - delta[(size_t)c * nchan + r] : delta[(size_t)r * nchan + c];
  }
};

// A block of 256 threads takes 64 input rows (c, one per lane) of row tile rt, each wave
// of it a fourth of the tile's waves: a thread's loads of the delay matrix are what a
// build waits for.
constexpr int kCols = 64, kSlices = 4;
struct Column {
  int dmin[kSlices][kCols], need[kSlices][kCols];
};

// The wave entries of this thread's waves; returns why they do not fit the variant, or
// 0, what the waves need staged, and how many of them follow no row pattern.
__device__ int table_waves(const Variant& v, const DelayView& delay, int rows_out, int rows_in, int rt, int c, int sbase,
                           int32_t* wav, int& need, int& plain) {
  const int DT = v.nwave * v.dpw, WI = v.wav_ints();
  // rows past the end repeat the last row (their results are not stored)
  auto d = [&](int k) { return delay(min(rt * DT + k, rows_out - 1), c); };
  for (int w = threadIdx.x / kCols; w < v.nwave; w += kSlices) {
    int32_t* e = wav ? wav + (((size_t)rt * v.nwave + w) * rows_in + c) * WI : nullptr;
    if (v.kind == KIND_WIN_F32) {
      int wmin = d(w * v.dpw);
      for (int j = 1; j < v.dpw; ++j) wmin = min(wmin, d(w * v.dpw + j));
      const int ws = (wmin - sbase) & ~3;
      if (ws > v.rowcap) return kTablesRow;
      int maxo = 0;
      if (v.jmp == 3) {
        // row blocks: the offsets' pattern if it has a block, else the slots (target 0)
        int m = INT32_MAX, top = 0, prev = 0, p = 0, packed = 0;
        for (int j = 0; j < v.dpw; ++j) {
          const int o = d(w * v.dpw + j) - sbase - ws;
          if (o < 0 || o > v.nwin - v.tp) return kTablesWindow;
          maxo = max(maxo, o);
          packed |= o << (8 * j);
          if (j > 0) {
            m = min(m, o - prev);
            top = max(top, o - prev);
          }
          prev = o;
        }
        const int nl = max(v.tp / 4 + 1, (v.tp + maxo + 3) / 4);
        need = max(need, ws + 63 * v.tp + 4 * nl);
        const int o0 = packed & 0xff;
        const bool pattern = m >= 0 && top - m <= 1 && m < v.row_classes() && o0 < 4;
        plain += pattern ? 0 : 1;
        if (!e) continue;
        const bool last = c % v.cc == v.cc - 1 || c == rows_in - 1;
        int target = 0;
        if (!last && pattern) {
          for (int j = 1; j < v.dpw; ++j)
            p |= ((packed >> (8 * j) & 0xff) - (packed >> (8 * j - 8) & 0xff) - m) << (j - 1);
          target = v.row_block(m, p, o0);
        }
        // reads beyond those the row before asks for (as many as its last offset needs)
        int extra = 0;
        if (c > 0) {
          auto d1 = [&](int j) { return delay(min(rt * DT + w * v.dpw + j, rows_out - 1), c - 1); };
          int pmin = d1(0);
          for (int j = 1; j < v.dpw; ++j) pmin = min(pmin, d1(j));
          const int olast = d1(v.dpw - 1) - (pmin & ~3);
          if (nl > min(v.nwin / 4, max(v.tp / 4 + 1, (v.tp + olast + 3) / 4))) extra = nl;
        }
        e[0] = 4 * ws;
        e[1] = target;
        e[2] = packed;
        e[3] = nl | extra << 8 | (last ? 0 : (int)0x80000000u);
        continue;
      }
      for (int j = 0; j < v.dpw; ++j) {
        const int o = d(w * v.dpw + j) - sbase - ws;
        if (o < 0 || o > v.nwin - v.tp) return kTablesWindow;
        maxo = max(maxo, o);
        if (e) e[2 + j] = v.jmp ? o * (v.prefetch() && j == v.dpw - 1 ? v.last_stride() : 4 * v.tp + 4) : o;
      }
      const int nl = max(v.tp / 4 + 1, (v.tp + maxo + 3) / 4);
      if (e) {
        for (int j = 2 + v.dpw; j < WI; ++j) e[j] = 0;
        e[0] = ws;
        e[1] = nl;
        if (v.prefetch() && c > 0) {
          // reads beyond those the row before already asked for (as many as its last slot needed)
          auto d1 = [&](int j) { return delay(min(rt * DT + w * v.dpw + j, rows_out - 1), c - 1); };
          int pmin = d1(0);
          for (int j = 1; j < v.dpw; ++j) pmin = min(pmin, d1(j));
          const int olast = d1(v.dpw - 1) - (pmin & ~3);
          const int asked = min(v.nwin / 4, max(v.tp / 4 + 1, (v.tp + olast + 3) / 4));
          e[6] = nl > asked ? nl : 0;
        }
      }
      // full-window variants read all nwin samples of every row
      need = max(need, ws + 63 * v.tp + (v.jmp == 2 ? v.nwin : 4 * nl));
    } else if (v.kind == KIND_LANE_F32) {
      for (int j = 0; j < v.dpw; ++j) {
        const int o = d(w * v.dpw + j) - sbase;
        if (o > v.rowcap) return kTablesRow;
        if (e) e[j] = 4 * (c % v.cc * v.rowcap + o);  // byte offset in the pass's buffer
        need = max(need, o + 64 * v.tp);
      }
    } else {
      uint32_t packed[4] = {0, 0, 0, 0};
      for (int j = 0; j < v.dpw; ++j) {
        const int o = d(w * v.dpw + j) - sbase;
        if (o > 65535) return kTablesOffset;
        if (v.mode == 0)
          packed[j >> 1] |= (uint32_t)o << (16 * (j & 1));
        else if (e)
          // byte offset into the staged copies: copy o & 3, row slot c % cc, dword o >> 2
          e[j] = 4 * (((o & 3) * v.cc + c % v.cc) * (v.rowcap / 4) + (o >> 2));
        need = max(need, (o & ~3) + 256 * v.tp + 4);
      }
      if (e && v.mode == 0)
        for (int j = 0; j < WI; ++j) e[j] = (int32_t)packed[j];
      else if (e)
        for (int j = v.dpw; j < WI; ++j) e[j] = 0;
    }
  }
  return 0;
}

// The tables' entries of input row c for row tile rt (not written when blk and wav are
// null); returns why they do not fit the variant, or 0 (see table_waves).  Every thread of the block calls it.
__device__ int table_columns(const Variant& v, const DelayView& delay, int rows_out, int rows_in, int rt, int c,
                             int32_t* blk, int32_t* wav, int& plain) {
  __shared__ Column col;
  const int lane = threadIdx.x % kCols, slice = threadIdx.x / kCols;
  const bool live = c < rows_in;
  int dmin = INT32_MAX;
  if (live)
    for (int k = slice; k < v.dt(); k += kSlices) dmin = min(dmin, delay(min(rt * v.dt() + k, rows_out - 1), c));
  col.dmin[slice][lane] = dmin;
  __syncthreads();
  for (int s = 0; s < kSlices; ++s) dmin = min(dmin, col.dmin[s][lane]);
  const int sbase = v.kind == KIND_TILE_U8 ? dmin & ~15 : dmin & ~3;
  int need = 0;
  int why = live ? table_waves(v, delay, rows_out, rows_in, rt, c, sbase, wav, need, plain) : 0;
  col.need[slice][lane] = need;
  __syncthreads();
  for (int s = 0; s < kSlices; ++s) need = max(need, col.need[s][lane]);
  const int unit = v.kind == KIND_TILE_U8 ? 16 : 4;
  need = (need + unit - 1) / unit * unit;
  if (need > v.rowcap) why = max(why, (int)kTablesRow);
  if (blk && live && slice == 0) {
    blk[((size_t)rt * rows_in + c) * 2 + 0] = sbase;
    blk[((size_t)rt * rows_in + c) * 2 + 1] = need;
  }
  return why;
}

// One variant per blockIdx.y, each with its own number of row tiles.
struct BuildList {
  TableBuild b[kFitBatch];
};
__global__ __launch_bounds__(256) void build_tables_kernel(BuildList list, DelayView delay, int rows_out, int rows_in) {
  const TableBuild& b = list.b[blockIdx.y];
  const int ncb = (rows_in + kCols - 1) / kCols;
  const int rt = blockIdx.x / ncb;
  const int c = (blockIdx.x - rt * ncb) * kCols + threadIdx.x % kCols;
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k < b.slack; k += 256) b.wav[b.ent + k] = 0;
  int plain = 0;
  if (rt * b.v.dt() < rows_out) (void)table_columns(b.v, delay, rows_out, rows_in, rt, c, b.blk, b.wav, plain);
}

// Whether the variants fit: bad[k] (zero before) becomes the reason if variant k does not;
// bad[kFitBatch + k] counts the wave entries that follow no row pattern.
struct VariantList {
  Variant v[kFitBatch];
};
__global__ __launch_bounds__(256) void check_fits_kernel(VariantList list, DelayView delay, int rows_out, int rows_in,
                                                         int* bad) {
  const Variant& v = list.v[blockIdx.y];
  const int ncb = (rows_in + kCols - 1) / kCols;
  const int rt = blockIdx.x / ncb;
  const int c = (blockIdx.x - rt * ncb) * kCols + threadIdx.x % kCols;
  if (rt * v.dt() >= rows_out) return;
  int plain = 0;
  const int why = table_columns(v, delay, rows_out, rows_in, rt, c, nullptr, nullptr, plain);
  if (why) atomicMax(bad + blockIdx.y, why);
  if (plain) atomicAdd(bad + kFitBatch + blockIdx.y, plain);
}

// Adjoint: per (row tile, pass) the least start and greatest end of the
// pass's staged windows.
__global__ __launch_bounds__(256) void build_span_kernel(BuildList list, int rows_out, int rows_in) {
  const TableBuild& b = list.b[blockIdx.y];
  const int cc = b.v.cc, npass = (rows_in + cc - 1) / cc;
  const int nqb = (npass + 255) / 256;
  const int rt = blockIdx.x / nqb;
  const int q = (blockIdx.x - rt * nqb) * 256 + threadIdx.x;
  if (rt * b.v.dt() >= rows_out || q >= npass) return;
  int smin = INT32_MAX, emax = INT32_MIN;
  for (int c = q * cc; c < min(rows_in, (q + 1) * cc); ++c) {
    const int32_t* e = b.blk + ((size_t)rt * rows_in + c) * 2;
    smin = min(smin, e[0]);
    emax = max(emax, e[0] + e[1]);
  }
  b.span[((size_t)rt * npass + q) * 2 + 0] = smin;
  b.span[((size_t)rt * npass + q) * 2 + 1] = emax;
}

}  // namespace

hipError_t launch_build_tables(const std::vector<TableBuild>& bs, const int32_t* d_delay, int nchan, int ndm,
                               bool adjoint, int pad, hipStream_t s) {
  if (bs.empty() || bs.size() > kFitBatch) return hipErrorInvalidValue;
  const int rows_out = adjoint ? nchan : ndm, rows_in = adjoint ? ndm : nchan;
  BuildList list = {};
  int64_t grid = 0, sgrid = 0;
  for (size_t k = 0; k < bs.size(); ++k) {
    const Variant& v = bs[k].v;
    const int64_t nrt = (rows_out + v.dt() - 1) / v.dt();
    list.b[k] = bs[k];
    grid = std::max(grid, nrt * ((rows_in + kCols - 1) / kCols));
    sgrid = std::max(sgrid, nrt * (((rows_in + v.cc - 1) / v.cc + 255) / 256));
  }
  if (grid > 0x7fffffff) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(build_tables_kernel, dim3((unsigned)grid, (unsigned)bs.size()), dim3(256), 0, s, list,
                     DelayView{d_delay, nchan, adjoint, pad}, rows_out, rows_in);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && adjoint) {
    hipLaunchKernelGGL(build_span_kernel, dim3((unsigned)sgrid, (unsigned)bs.size()), dim3(256), 0, s, list, rows_out,
                       rows_in);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_check_fits(const std::vector<const Variant*>& vs, const int32_t* d_delay, int nchan, int ndm,
                             bool adjoint, int pad, int* bad, hipStream_t s) {
  if (vs.empty() || vs.size() > kFitBatch) return hipErrorInvalidValue;
  const int rows_out = adjoint ? nchan : ndm, rows_in = adjoint ? ndm : nchan;
  VariantList list = {};
  int64_t nrt = 1;
  for (size_t k = 0; k < vs.size(); ++k) {
    list.v[k] = *vs[k];
    nrt = std::max<int64_t>(nrt, (rows_out + vs[k]->dt() - 1) / vs[k]->dt());
  }
  const int64_t grid = nrt * ((rows_in + kCols - 1) / kCols);
  if (grid > 0x7fffffff) return hipErrorInvalidConfiguration;
  hipError_t e = hipMemsetAsync(bad, 0, 2 * kFitBatch * sizeof(int), s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(check_fits_kernel, dim3((unsigned)grid, (unsigned)vs.size()), dim3(256), 0, s, list,
                     DelayView{d_delay, nchan, adjoint, pad}, rows_out, rows_in, bad);
  return hipGetLastError();
}

}  // namespace dd
