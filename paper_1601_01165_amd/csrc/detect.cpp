// Host side of the single-pulse search (boxcar S/N over every dedispersed
// series, the detection step of the real-time pipeline of Section 1): the
// fused path runs a tile kernel whose epilogue searches the tile instead of
// storing it, then merges the per-tile records; the unfused path searches
// stored rows.  The definition is documented with dedisp_detect.
#include <algorithm>
#include <string>

#include "internal.h"

namespace dd {
dedisp_status ensure_tables(dedisp_plan p, int dir, int vi, Tables** out);

// Keys of the uint8 search hold (window sum << IB) in 31 bits: prefix sums over
// a lane's run and look-ahead must stay below 2^30.
static bool u8_sums_fit(const Variant& v, int nchan) {
  const int run = 4 * v.tp;
  const double scale = (double)run;  // 2^IB == run
  return (double)(run + kDetLook - 1) * 255.0 * nchan * scale < (double)(1 << 30);
}

static bool det_fits(dedisp_plan p, bool u8, int vi) {
  const std::vector<Variant>& vs = u8 ? variants_u8() : variants_f32();
  if (vi < 0 || vi >= (int)vs.size()) return false;
  const Variant& v = vs[vi];
  if (!detect_fusable(v)) return false;
  if (u8 && !u8_sums_fit(v, p->nchan)) return false;
  return ensure_tables(p, u8 ? 1 : 0, vi, nullptr) == DEDISP_OK;
}

// The variant of the search for this plan and dtype: the one set or tuned
// (-1: unfused), otherwise the automatic choice.
//   float32: unfused.  Storing the series and searching them costs about 0.05 ms
//     on the 1024-channel, 2000-DM beam; the fused forms lose more by their
//     registers and overlapping tiles (1.10 ms unfused, 1.27 ms the best fused).  On few
//     channels the series cost more than the sums (8 beams of 22 channels, 2121 DM
//     trials, 11,614 samples: 606 us unfused, 366 fused), and where one beam's series
//     take more than 1 GiB, the memory: fused then, if a variant fits (search_path).
//   uint8: the first that fits from a preference list (fastest first on the
//     32-channel, 2048-DM beam: the int32 series would be 1.64 GB), or with
//     fewer blocks than CUs the same kernel with half the samples per tile
//     (29 channels, 131 DM trials, 20,011 samples: 21.9 against 26.9 us).
// What it takes is noted in the plan, so that the tables stay when others are dropped.
static int automatic(dedisp_plan p, bool u8, int vi) {
  std::vector<int>& ids = p->det_auto[u8];
  if (std::find(ids.begin(), ids.end(), vi) == ids.end()) ids.push_back(vi);
  return vi;
}

static constexpr int kDetSmallTile = 25;  // 32 DMs x 512 of the 32 DMs x 1024 of variant 23

static int det_variant(dedisp_plan p, bool u8) {
  const int set = u8 ? p->var_det_u8 : p->var_det_f32;
  if (set >= -1) return set;
  if (!u8) return -1;
  static const int pref_u8[] = {23, 14, 25, 27, 16, 15, 12, 17, 18, 20, 13, 21, 19, 24, 26};
  for (int vi : pref_u8)
    if (det_fits(p, true, vi)) return automatic(p, true, vi);
  return -1;
}

static size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

static int64_t rows_tiles(int nsamp) { return (nsamp + kDetRowsStep - 1) / kDetRowsStep; }

static size_t rows_ws(int64_t nrows, int nsamp) { return (size_t)nrows * rows_tiles(nsamp) * sizeof(DetRec); }

// Records of a fused search.
static size_t fused_ws(dedisp_plan p, const Variant& v, int nbeam, int nsamp) {
  return (size_t)nbeam * p->ndm * ((nsamp + det_step(v) - 1) / det_step(v)) * sizeof(DetRec);
}

// Unfused path: the forward map of some beams into the workspace, then the row
// search.  Beams go through it in groups whose series and records take at most
// 1 GiB (one beam at least), fewer at a time in a smaller workspace.
static constexpr size_t kUnfusedBytes = (size_t)1 << 30;
static constexpr size_t kUnfusedSlack = 256;  // the records start on the next multiple of this

static size_t beam_series(dedisp_plan p, int nsamp) { return (size_t)p->ndm * round_up(nsamp, 4) * 4; }

static size_t unfused_beam_ws(dedisp_plan p, int nsamp) {
  return beam_series(p, nsamp) + (size_t)p->ndm * rows_tiles(nsamp) * sizeof(DetRec);
}

static size_t unfused_ws(dedisp_plan p, int nbeam, int nsamp) {
  const size_t beam = unfused_beam_ws(p, nsamp);
  return std::min(nbeam * beam, std::max(kUnfusedBytes, beam)) + kUnfusedSlack;
}

// Beams per group in a workspace of ws_bytes; 0: not even one fits.
static int unfused_beams(dedisp_plan p, int nbeam, int nsamp, size_t ws_bytes) {
  const size_t beam = unfused_beam_ws(p, nsamp);
  if (ws_bytes < kUnfusedSlack + beam) return 0;
  const size_t most = std::max<size_t>(1, kUnfusedBytes / beam);
  return (int)std::min({(size_t)nbeam, most, (ws_bytes - kUnfusedSlack) / beam});
}

// Few channels: below this many the fused search is the faster from this much of
// series on (us, fused and unfused: 8 beams of 22 channels, 2121 DM trials, 11,614 samples 366
// and 606; 48 channels, 4 beams of 1000 DM trials, 20,000 samples 219 and 278; 16 channels, 100 DM
// trials, 5000 samples 22 and 11; 85 channels, 3 beams of 348 DM trials, 9591 samples 69 and 57.
// Over 108 random calls of 8 to 63 channels, 4 to 300 DM trials 1.1 times as fast as unfused
// on average, 0.84 to 1.6).  Tiles of more than 16 DM trials (delay spans too wide for the
// first of `few`) need two of them for that: 39's 48 leave most of their waves without work on
// 12 DM trials (40 beams of 45 channels, 53,352 samples: 254 us, 137 unfused), and are
// 0.78 to 0.99 times as fast up to 79 DM trials, 0.91 to 1.25 from 97.
static constexpr int kFewChannels = 64;
static constexpr size_t kFewBytes = (size_t)32 << 20;

// The variant that searches float32 beams in place, or -1.
static int f32_in_place(dedisp_plan p) {
  static const int few[] = {20, 16, 14, 18, 13, 15, 17, 39}, many[] = {42, 41, 39, 16, 14, 18, 13, 15, 17};
  if (p->nchan < kFewChannels) {
    for (int k : few)
      if (det_fits(p, false, k)) return automatic(p, false, k);
  } else {
    for (int k : many)
      if (det_fits(p, false, k)) return automatic(p, false, k);
  }
  return -1;
}

// Whether float32 calls of these sizes go in place if they can.
static bool f32_prefers_in_place(dedisp_plan p, int nbeam, int nsamp) {
  const size_t beam = beam_series(p, nsamp);
  if (beam > kUnfusedBytes) return true;
  if (p->nchan >= kFewChannels || nbeam * beam <= kFewBytes) return false;
  const int k = f32_in_place(p);
  if (k < 0) return false;
  const int dt = variants_f32()[k].dt();
  return dt <= 16 || p->ndm >= 2 * dt;
}

// uint8: the small tile beside the default variant vi, or -1.  Looked at on the
// first call whatever its size, so that later ones allocate nothing.
static int u8_small_tile(dedisp_plan p, int vi) {
  if (vi < 0 || vi == kDetSmallTile || p->var_det_u8 >= -1 || !det_fits(p, true, kDetSmallTile)) return -1;
  return automatic(p, true, kDetSmallTile);
}

// The path of a call with a workspace of ws_bytes: a fused variant, or -1 and the
// beams per group.  False if the workspace serves none.  A workspace sized
// (search_ws) for a call serves every call with no more beams and no more samples.
static bool search_path(dedisp_plan p, bool u8, int nbeam, int nsamp, size_t ws_bytes, int& vi, int& beams) {
  const std::vector<Variant>& vs = u8 ? variants_u8() : variants_f32();
  vi = det_variant(p, u8);
  beams = 0;
  if (u8) {
    const int small = u8_small_tile(p, vi);
    if (small >= 0) {
      const Variant& v = vs[vi];
      const int64_t blocks = (int64_t)((p->ndm + v.dt() - 1) / v.dt()) * ((nsamp + det_step(v) - 1) / det_step(v)) * nbeam;
      if (blocks < p->ncu && ws_bytes >= fused_ws(p, vs[small], nbeam, nsamp)) vi = small;
    }
  } else if (vi < 0 && p->var_det_f32 < -1) {
    // in place too where the workspace (sized for such a call) is too small for one beam's series
    if (f32_prefers_in_place(p, nbeam, nsamp) || unfused_beams(p, nbeam, nsamp, ws_bytes) == 0) vi = f32_in_place(p);
  }
  if (vi >= 0) return ws_bytes >= fused_ws(p, vs[vi], nbeam, nsamp);
  beams = unfused_beams(p, nbeam, nsamp, ws_bytes);
  return beams > 0;
}

static size_t search_ws(dedisp_plan p, bool u8, int nbeam, int nsamp) {
  const std::vector<Variant>& vs = u8 ? variants_u8() : variants_f32();
  int vi = det_variant(p, u8);
  size_t n = 0;
  if (!u8 && vi < 0 && p->var_det_f32 < -1 && f32_prefers_in_place(p, nbeam, nsamp)) {
    vi = f32_in_place(p);
    // few channels: room for the series too, which a smaller call stores
    if (beam_series(p, nsamp) <= kUnfusedBytes) n = unfused_ws(p, nbeam, nsamp);
  }
  if (vi < 0) return unfused_ws(p, nbeam, nsamp);
  n = std::max(n, fused_ws(p, vs[vi], nbeam, nsamp));
  const int small = u8 ? u8_small_tile(p, vi) : -1;
  if (small >= 0) {
    // The small tile's records too, as far as a call with fewer blocks than CUs can need
    // them: row tiles x time tiles x beams < CUs, each time tile cut into `cut`.
    const Variant& v = vs[vi];
    const int64_t tiles = (p->ncu - 1) / ((p->ndm + v.dt() - 1) / v.dt());
    const int64_t cut = (det_step(v) + det_step(vs[small]) - 1) / det_step(vs[small]);
    n = std::max(n, std::min(fused_ws(p, vs[small], nbeam, nsamp), (size_t)(tiles * cut) * p->ndm * sizeof(DetRec)));
  }
  return n;
}

}  // namespace dd

using namespace dd;

extern "C" {

size_t dedisp_detect_workspace_bytes(dedisp_plan p, dedisp_dtype in_type, int32_t nbeam, int32_t nsamp) {
  if (!p || nbeam < 1 || nsamp < 1 || (in_type != DEDISP_F32 && in_type != DEDISP_U8)) return 0;
  const bool u8 = in_type == DEDISP_U8;
  const size_t n = search_ws(p, u8, nbeam, nsamp);
  // the forward kernels' tables, so that a search with this workspace allocates nothing
  if (det_variant(p, u8) < 0) (void)dedisp_plan_prepare(p, in_type, 0);
  return n;
}

int32_t dedisp_detect_variant(dedisp_plan p, dedisp_dtype in_type) {
  if (!p || (in_type != DEDISP_F32 && in_type != DEDISP_U8)) return -1;
  return det_variant(p, in_type == DEDISP_U8);
}

static dedisp_status check_outputs(int32_t nwidth, const double* d_snr, const int32_t* d_width,
                                   const int32_t* d_start) {
  if (nwidth < 1 || nwidth > kDetNW) return fail(DEDISP_E_INVALID, "nwidth must be in [1, 6]");
  if (!d_snr || !d_width || !d_start) return fail(DEDISP_E_INVALID, "snr, width and start must not be NULL");
  return DEDISP_OK;
}

dedisp_status dedisp_detect(dedisp_plan p, int32_t nbeam, int32_t nsamp, const void* d_in, dedisp_dtype in_type,
                            int64_t in_stride, const float* d_w, int32_t nwidth, double* d_snr, int32_t* d_width,
                            int32_t* d_start, double* d_mean, double* d_std, void* d_ws, size_t ws_bytes,
                            void* stream) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (nbeam < 1 || nsamp < 1) return fail(DEDISP_E_INVALID, "nbeam and nsamp must be >= 1");
  if (nbeam > kMaxBeams) return fail(DEDISP_E_SHAPE, "at most 65535 beams per call");
  if (!d_in) return fail(DEDISP_E_INVALID, "input pointer is NULL");
  dedisp_status st = check_outputs(nwidth, d_snr, d_width, d_start);
  if (st != DEDISP_OK) return st;
  const bool u8 = in_type == DEDISP_U8;
  if (!u8 && in_type != DEDISP_F32) return fail(DEDISP_E_DTYPE, "input must be F32 or U8");
  if (u8 && d_w) return fail(DEDISP_E_DTYPE, "weights are not supported for uint8 input");
  if (in_stride < (int64_t)nsamp + p->max_delay) return fail(DEDISP_E_SHAPE, "in_stride < nsamp + max_delay");
  if (in_stride > kMaxRow || (int64_t)nsamp + p->max_delay > kMaxRow)
    return fail(DEDISP_E_SHAPE, "rows longer than 2^29 samples are not supported");
  const int esz = u8 ? 1 : 4;
  if (((uintptr_t)d_in & 15u) || (in_stride * esz) % 16 || (d_w && ((uintptr_t)d_w & 3)))
    return fail(DEDISP_E_ALIGN, "pointers and row byte sizes must be multiples of 16 bytes");
  if (!d_ws) return fail(DEDISP_E_WORKSPACE, "workspace is NULL");
  int vi, beams;
  if (!search_path(p, u8, nbeam, nsamp, ws_bytes, vi, beams)) return fail(DEDISP_E_WORKSPACE, "workspace too small");
  if ((uintptr_t)d_ws & 15u) return fail(DEDISP_E_ALIGN, "workspace must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int64_t nseries = (int64_t)nbeam * p->ndm;
  if (nseries > 0x7ffffff0) return fail(DEDISP_E_SHAPE, "too many series");
  hipError_t e;
  if (vi < 0) {
    const int64_t stride = round_up(nsamp, 4);
    void* rows = d_ws;
    DetRec* recs = (DetRec*)((char*)d_ws + round_up((size_t)beams * p->ndm * stride * 4, kUnfusedSlack));
    const int ntiles = (int)rows_tiles(nsamp);
    for (int b = 0; b < nbeam; b += beams) {
      const int nb = std::min(beams, nbeam - b);
      const int64_t s0 = (int64_t)b * p->ndm;
      st = dedisp_execute(p, nb, nsamp, (const char*)d_in + (int64_t)b * p->nchan * in_stride * esz, in_type, in_stride,
                          d_w, rows, u8 ? DEDISP_I32 : DEDISP_F32, stride, stream);
      if (st != DEDISP_OK) return st;
      e = launch_detect_rows(rows, u8, stride, nb * p->ndm, nsamp, ntiles, nwidth, recs, d_snr + s0, d_width + s0,
                             d_start + s0, d_mean ? d_mean + s0 : nullptr, d_std ? d_std + s0 : nullptr, s);
      if (e != hipSuccess) return hip_fail(e, "launching the row search");
    }
    return DEDISP_OK;
  }
  Tables* t = nullptr;
  st = ensure_tables(p, u8 ? 1 : 0, vi, &t);
  if (st != DEDISP_OK) return st;
  const Variant& v = (u8 ? variants_u8() : variants_f32())[vi];
  const int step = det_step(v);
  TileArgs a = {};
  a.in = d_in;
  a.in_stride = in_stride;
  a.in_beam_stride = in_stride * p->nchan;
  a.in_shift = 0;
  a.in_lo = 0;
  a.in_hi = (int)in_stride;
  a.rows_in = p->nchan;
  a.rows_out = p->ndm;
  a.nout = nsamp;
  a.n_time_tiles = (nsamp + step - 1) / step;
  a.n_row_tiles = t->n_row_tiles;
  a.tiles_per_block = 1;
  a.blk = t->d_blk;
  a.wav = t->d_wav;
  a.w_in = d_w;
  a.out = nullptr;
  a.tile_step = step;
  a.det_nsamp = nsamp;
  // a lane's sum of squares in 32 bits: run * (255 * nchan)^2 < 2^32
  a.det_s2_u32 = u8 && (double)(4 * v.tp) * (255.0 * p->nchan) * (255.0 * p->nchan) < 4294967296.0;
  a.det = (DetRec*)d_ws;
  e = launch_detect(v, a, nbeam, s);
  if (e != hipSuccess) return hip_fail(e, "launching the fused search");
  e = launch_det_finish(a.det, u8, (int)nseries, a.n_time_tiles, nsamp, nwidth, d_snr, d_width, d_start, d_mean,
                        d_std, s);
  return e == hipSuccess ? DEDISP_OK : hip_fail(e, "launching the record merge");
}

dedisp_status dedisp_plan_set_detect_variant(dedisp_plan p, dedisp_dtype in_type, int32_t vi) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (in_type != DEDISP_F32 && in_type != DEDISP_U8) return fail(DEDISP_E_DTYPE, "dtype must be F32 or U8");
  const bool u8 = in_type == DEDISP_U8;
  const int n = (int)(u8 ? variants_u8() : variants_f32()).size();
  if (vi < -2 || vi >= n) return fail(DEDISP_E_INVALID, "variant index out of range");
  if (vi >= 0 && !det_fits(p, u8, vi)) return fail(DEDISP_E_UNTUNED, "variant has no search epilogue or does not fit");
  (u8 ? p->var_det_u8 : p->var_det_f32) = vi;
  return DEDISP_OK;
}

dedisp_status dedisp_detect_autotune(dedisp_plan p, int32_t nbeam, int32_t nsamp, dedisp_dtype in_type, int32_t nwidth,
                                     float* ms, int32_t n) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (nbeam < 1 || nsamp < 1) return fail(DEDISP_E_INVALID, "nbeam and nsamp must be >= 1");
  if (in_type != DEDISP_F32 && in_type != DEDISP_U8) return fail(DEDISP_E_DTYPE, "dtype must be F32 or U8");
  if (nwidth < 1 || nwidth > kDetNW) return fail(DEDISP_E_INVALID, "nwidth must be in [1, 6]");
  const bool u8 = in_type == DEDISP_U8;
  const int nv = (int)(u8 ? variants_u8() : variants_f32()).size();
  const int esz = u8 ? 1 : 4;
  const int64_t q = 16 / esz;
  const int64_t in_stride = ((int64_t)nsamp + p->max_delay + q - 1) / q * q;
  const int64_t nseries = (int64_t)nbeam * p->ndm;
  // room for every path: the series of a few beams, or the records of all of them (64
  // bytes per series and tile: more than 1 GiB from about 30 GiB of series on)
  size_t ws_bytes = unfused_ws(p, nbeam, nsamp);
  for (int vi = 0; vi < nv; ++vi)
    if (det_fits(p, u8, vi))
      ws_bytes = std::max(ws_bytes, fused_ws(p, (u8 ? variants_u8() : variants_f32())[vi], nbeam, nsamp));
  void *d_in = nullptr, *d_ws = nullptr, *d_res = nullptr;
  hipError_t e = hipMalloc(&d_in, (size_t)nbeam * p->nchan * in_stride * esz);
  if (e == hipSuccess) e = hipMalloc(&d_ws, ws_bytes);
  if (e == hipSuccess) e = hipMalloc(&d_res, (size_t)nseries * 16);
  if (e == hipSuccess) e = launch_fill_random(d_in, (size_t)nbeam * p->nchan * in_stride * esz, !u8, 1601u, nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    if (d_in) (void)hipFree(d_in);
    if (d_ws) (void)hipFree(d_ws);
    if (d_res) (void)hipFree(d_res);
    return e == hipErrorOutOfMemory ? fail(DEDISP_E_NOMEM, "autotune scratch allocation failed")
                                    : hip_fail(e, "autotune scratch");
  }
  double* snr = (double*)d_res;
  int32_t* wid = (int32_t*)(snr + nseries);
  int32_t* start = wid + nseries;
  hipStream_t s;
  hipEvent_t e0, e1;
  (void)hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  (void)hipEventCreate(&e0);
  (void)hipEventCreate(&e1);
  int& var = u8 ? p->var_det_u8 : p->var_det_f32;
  const int saved = var;
  std::vector<float> times(nv + 1, -1.f);
  int best = -2;
  float best_ms = 1e30f;
  for (int vi = -1; vi < nv; ++vi) {
    if (vi >= 0 && !det_fits(p, u8, vi)) continue;
    var = vi;
    const float t = median_ms(
        [&]() {
          return dedisp_detect(p, nbeam, nsamp, d_in, in_type, in_stride, nullptr, nwidth, snr, wid, start, nullptr,
                               nullptr, d_ws, ws_bytes, s) == DEDISP_OK
                     ? hipSuccess
                     : hipErrorUnknown;
        },
        s, 3, e0, e1);
    times[vi < 0 ? nv : vi] = t;
    if (t > 0 && t < best_ms) {
      best_ms = t;
      best = vi;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipStreamDestroy(s);
  (void)hipFree(d_in);
  (void)hipFree(d_ws);
  (void)hipFree(d_res);
  if (ms)
    for (int i = 0; i < n && i <= nv; ++i) ms[i] = times[i];
  if (best == -2) {
    var = saved;
    return fail(DEDISP_E_UNTUNED, "no search path ran");
  }
  var = best;
  return DEDISP_OK;
}

size_t dedisp_detect_rows_workspace_bytes(int32_t nrows, int32_t nsamp) {
  if (nrows < 1 || nsamp < 1) return 0;
  return rows_ws(nrows, nsamp);
}

dedisp_status dedisp_detect_rows(int32_t nrows, int32_t nsamp, const void* d_rows, dedisp_dtype type, int64_t stride,
                                 int32_t nwidth, double* d_snr, int32_t* d_width, int32_t* d_start, double* d_mean,
                                 double* d_std, void* d_ws, size_t ws_bytes, void* stream) {
  if (nrows < 1 || nsamp < 1) return fail(DEDISP_E_INVALID, "nrows and nsamp must be >= 1");
  if (!d_rows) return fail(DEDISP_E_INVALID, "rows pointer is NULL");
  dedisp_status st = check_outputs(nwidth, d_snr, d_width, d_start);
  if (st != DEDISP_OK) return st;
  if (type != DEDISP_F32 && type != DEDISP_I32) return fail(DEDISP_E_DTYPE, "rows must be F32 or I32");
  if (stride < nsamp) return fail(DEDISP_E_SHAPE, "stride < nsamp");
  if (stride > kMaxRow) return fail(DEDISP_E_SHAPE, "rows longer than 2^29 samples are not supported");
  if (((uintptr_t)d_rows & 15u) || (stride * 4) % 16)
    return fail(DEDISP_E_ALIGN, "pointers and row byte sizes must be multiples of 16 bytes");
  if (!d_ws) return fail(DEDISP_E_WORKSPACE, "workspace is NULL");
  if ((uintptr_t)d_ws & 15u) return fail(DEDISP_E_ALIGN, "workspace must be 16-byte aligned");
  if (ws_bytes < rows_ws(nrows, nsamp)) return fail(DEDISP_E_WORKSPACE, "workspace too small");
  hipStream_t s = (hipStream_t)stream;
  const int ntiles = (int)rows_tiles(nsamp);
  DetRec* recs = (DetRec*)d_ws;
  const hipError_t e = launch_detect_rows(d_rows, type == DEDISP_I32, stride, nrows, nsamp, ntiles, nwidth, recs, d_snr,
                                          d_width, d_start, d_mean, d_std, s);
  return e == hipSuccess ? DEDISP_OK : hip_fail(e, "launching the row search");
}

}  // extern "C"
