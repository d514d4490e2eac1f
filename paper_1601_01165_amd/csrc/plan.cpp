// Host side of the dedispersion library: plans, delay tables, tile tables,
// argument validation and the forward / adjoint entry points of the C-ABI.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <climits>
#include <cstdio>
#include <functional>
#include <map>
#include <mutex>
#include <limits>
#include <new>
#include <string>
#include <vector>

#include "internal.h"

namespace dd {

static thread_local std::string g_last_error;

dedisp_status fail(dedisp_status st, const std::string& msg) {
  g_last_error = msg;
  return st;
}

dedisp_status hip_fail(hipError_t e, const char* what) {
  g_last_error = std::string(what) + ": " + hipGetErrorString(e);
  return DEDISP_E_HIP;
}

// ---------------------------------------------------------------------------
// Delay table (Section 2, Equation 1; computed ahead of time, Section 2.1).
//   f_h = highest channel frequency
//   k   = 4150 * DM * (1/f^2 - 1/f_h^2) seconds, f in MHz
//   delta = floor(k / tsamp + 1/2)
// ---------------------------------------------------------------------------
static dedisp_status build_delay_table(int nchan, const double* f, double tsamp, int ndm, const double* dm,
                                       std::vector<int32_t>& out, int& max_delay) {
  double fh = f[0];
  for (int c = 0; c < nchan; ++c) {
    if (!(f[c] > 0.0) || !std::isfinite(f[c])) return fail(DEDISP_E_INVALID, "channel frequency must be > 0 and finite");
    fh = std::max(fh, f[c]);
  }
  const double inv_fh2 = 1.0 / (fh * fh);
  out.assign((size_t)nchan * ndm, 0);
  max_delay = 0;
  for (int j = 0; j < ndm; ++j) {
    if (!(dm[j] >= 0.0) || !std::isfinite(dm[j])) return fail(DEDISP_E_INVALID, "DM must be >= 0 and finite");
    for (int c = 0; c < nchan; ++c) {
      const double kdelay = 4150.0 * dm[j] * (1.0 / (f[c] * f[c]) - inv_fh2);
      const double x = std::floor(kdelay / tsamp + 0.5);
      if (!(x >= 0.0) || x > 2147483647.0) return fail(DEDISP_E_SHAPE, "a delay does not fit in int32");
      out[(size_t)j * nchan + c] = (int32_t)x;
      max_delay = std::max(max_delay, (int)x);
    }
  }
  return DEDISP_OK;
}

// Device memory that is freed with its last user.
static hipError_t shared_malloc(std::shared_ptr<void>& mem, size_t bytes) {
  void* ptr = nullptr;
  const hipError_t e = hipMalloc(&ptr, bytes);
  if (e == hipSuccess) mem = std::shared_ptr<void>(ptr, [](void* q) { (void)hipFree(q); });
  return e;
}

// Sizes (ints, each part a multiple of 256 bytes) of a variant's tables.
struct TableSizes {
  size_t blk, ent, slack, span;
  size_t total() const { return blk + ent + slack + span; }
};
static TableSizes table_sizes(dedisp_plan p, int dir, const Variant& v) {
  const bool adj = dir == 2;
  const size_t rows_out = adj ? p->nchan : p->ndm, rows_in = adj ? p->ndm : p->nchan;
  const size_t nrt = (rows_out + v.dt() - 1) / v.dt();
  auto whole = [](size_t n) { return (n + 63) / 64 * 64; };
  TableSizes s;
  s.blk = whole(nrt * rows_in * 2);
  s.ent = nrt * v.nwave * rows_in * v.wav_ints();
  s.slack = whole(s.ent + (size_t)v.cc * v.wav_ints()) - s.ent;  // a whole pass can be read after the last row
  // The adjoint's input rows (DM trials) reach outside the output gradient's
  // samples for part of the time tiles: the span of each pass's staged
  // windows lets the kernel skip passes that would add only zeros.
  s.span = adj ? whole(nrt * ((rows_in + v.cc - 1) / v.cc) * 2) : 0;
  return s;
}

void drop_spare_tables(dedisp_plan p, int dir, int keep) {
  std::map<int, Tables>& m = dir == 0 ? p->fwd_f32 : dir == 1 ? p->fwd_u8 : p->adj_f32;
  for (auto it = m.begin(); it != m.end();) {
    const int vi = it->first;
    auto in = [vi](const std::vector<int>& ids) { return std::find(ids.begin(), ids.end(), vi) != ids.end(); };
    const int det = dir == 0 ? p->var_det_f32 : p->var_det_u8;
    const bool search = dir < 2 && (det == -2 ? in(p->det_auto[dir]) : vi == det);
    const bool chosen = vi == keep || search || (p->by_size[dir] && in(p->fine[dir])) ||
                        vi == (dir == 0 ? p->var_f32 : dir == 1 ? p->var_u8 : p->var_adj);
    if (chosen || it->second.pins > 0) {
      ++it;
      continue;
    }
    it = m.erase(it);
  }
}

// Learn which of the variants fit the plan in direction `dir` (0 = forward f32,
// 1 = forward u8, 2 = adjoint f32), as many as possible in one launch.
static dedisp_status check_fits(dedisp_plan p, int dir, const std::vector<int>& ids) {
  const std::vector<Variant>& vs = dir == 1 ? variants_u8() : variants_f32();
  const int rows_in = dir == 2 ? p->ndm : p->nchan;
  std::vector<int> ask;
  for (int vi : ids) {
    if (p->fits[dir].count(vi)) continue;
    if (vs[vi].kind == KIND_TILE_U8 && vs[vi].mode == 1 && rows_in > 256)
      p->fits[dir][vi] = kTablesPacked;
    else
      ask.push_back(vi);
  }
  for (size_t k0 = 0; k0 < ask.size(); k0 += kFitBatch) {
    const size_t n = std::min<size_t>(kFitBatch, ask.size() - k0);
    std::vector<const Variant*> list;
    for (size_t k = 0; k < n; ++k) list.push_back(&vs[ask[k0 + k]]);
    int bad[2 * kFitBatch];
    hipError_t e = launch_check_fits(list, p->d_delay, p->nchan, p->ndm, dir == 2, p->adj_pad, p->d_bad, nullptr);
    if (e == hipSuccess) e = hipMemcpy(bad, p->d_bad, sizeof(bad), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "checking which kernels fit");
    for (size_t k = 0; k < n; ++k) {
      const Variant& v = *list[k];
      const double waves = ((dir == 2 ? p->nchan : p->ndm) + v.dpw - 1) / v.dpw;  // those with output rows
      p->fits[dir][v.id] = bad[k];
      p->plain[dir][v.id] = (float)((unsigned)bad[kFitBatch + k] / (waves * rows_in));
    }
  }
  return DEDISP_OK;
}

// Build the tables of the variants `ids` (each fits, none is built yet) in direction
// `dir` in one launch, complete for every stream on return.  Tables of 256 KiB and
// more lie in an allocation of their own, so that dropping them gives it back; smaller
// ones share one (an allocation costs more than building them).
static dedisp_status build_tables(dedisp_plan p, int dir, const std::vector<int>& ids) {
  std::map<int, Tables>& m = dir == 0 ? p->fwd_f32 : dir == 1 ? p->fwd_u8 : p->adj_f32;
  const std::vector<Variant>& vs = dir == 1 ? variants_u8() : variants_f32();
  constexpr size_t kOwn = (256 << 10) / sizeof(int32_t);
  size_t small = 0, at = 0;
  for (int vi : ids) {
    const size_t n = table_sizes(p, dir, vs[vi]).total();
    if (n < kOwn) small += n;
  }
  std::shared_ptr<void> common;
  hipError_t e = small ? shared_malloc(common, small * sizeof(int32_t)) : hipSuccess;
  std::vector<Tables> built;
  std::vector<TableBuild> bs;
  for (size_t k = 0; k < ids.size() && e == hipSuccess; ++k) {
    const Variant& v = vs[ids[k]];
    const TableSizes n = table_sizes(p, dir, v);
    Tables t;
    t.variant = ids[k];
    t.n_row_tiles = ((dir == 2 ? p->nchan : p->ndm) + v.dt() - 1) / v.dt();
    if (n.total() < kOwn) {
      t.mem = common;
      t.d_blk = static_cast<int32_t*>(common.get()) + at;
      at += n.total();
    } else {
      e = shared_malloc(t.mem, n.total() * sizeof(int32_t));
      t.d_blk = static_cast<int32_t*>(t.mem.get());
    }
    t.d_wav = t.d_blk + n.blk;
    if (n.span) t.d_span = t.d_wav + n.ent + n.slack;
    built.push_back(t);
    bs.push_back({v, t.d_blk, t.d_wav, t.d_span, n.ent, n.slack});
  }
  if (e != hipSuccess) return fail(DEDISP_E_NOMEM, "device allocation of tile tables failed");
  e = launch_build_tables(bs, p->d_delay, p->nchan, p->ndm, dir == 2, p->adj_pad, nullptr);
  if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  if (e != hipSuccess) return hip_fail(e, "building tile tables");
  for (const Tables& t : built) m.emplace(t.variant, t);
  return DEDISP_OK;
}

dedisp_status ensure_tables(dedisp_plan p, int dir, int vi, Tables** out) {
  std::map<int, Tables>& m = dir == 0 ? p->fwd_f32 : dir == 1 ? p->fwd_u8 : p->adj_f32;
  auto it = m.find(vi);
  if (it == m.end()) {
    const std::vector<Variant>& vs = dir == 1 ? variants_u8() : variants_f32();
    if (vi < 0 || vi >= (int)vs.size()) return fail(DEDISP_E_INVALID, "variant index out of range");
    dedisp_status st = check_fits(p, dir, {vi});
    if (st != DEDISP_OK) return st;
    static const char* const why[] = {"", "delay span within a wave exceeds the register window",
                                      "delay span within a block exceeds the LDS row",
                                      "delay span exceeds the 16-bit offset range",
                                      "more than 256 input rows overflow its packed sums"};
    if (p->fits[dir][vi]) return fail(DEDISP_E_UNTUNED, std::string(vs[vi].name) + ": " + why[p->fits[dir][vi]]);
    st = build_tables(p, dir, {vi});
    if (st != DEDISP_OK) return st;
    it = m.find(vi);
  }
  if (out) *out = &it->second;
  return DEDISP_OK;
}

// Variant preference when nothing was tuned, fastest first as measured on
// MI355X: forward FP32 on the 1024-channel, 2048-DM beam; forward uint8 on the
// 32-channel, 2048-DM beam (the packed sums of variant 22 take at most 256
// channels; past that the matrix-core shapes are 1.3 times as fast as the flushed
// packed sums, 1.06 against 1.41 ms on 1024 channels); the adjoint on 32 beams of
// 1024 channels and 1024 DMs.  The widest register windows and int32 sums come
// late: they fit the widest delay spans and the most channels.  In the adjoint
// the window of 84 comes right after those of 44: neighbouring channels differ by
// up to 12 samples on 1024 channels and 2048 DM trials, which only the
// 8-sample-per-lane forms took before (2.08 against 5.62 ms).
const std::vector<int>& default_order(int dir) {
  static const std::vector<int> f32 = {35, 34, 37, 38, 36, 32, 33, 22, 28, 21, 29, 31, 23, 30, 19, 20, 39, 40, 25, 24, 27, 26, 15, 18, 13,
                                       17, 9,  8,  16, 6,  14, 11, 7,  12, 10, 2,  3,  0,  1,  5,  4,  41, 42, 43, 46, 48, 45, 47, 44, 49, 50};
  static const std::vector<int> u8 = {22, 23, 25, 27, 26, 24, 16, 20, 15, 21, 12, 13, 17, 14, 18, 6, 2, 0, 5, 19, 9, 3, 4, 1, 8, 7, 10, 11};
  static const std::vector<int> adj = {37, 38, 39, 40, 26, 27, 32, 34, 35, 36, 33, 19, 21, 29, 20, 30, 9, 8, 6, 11, 12, 7, 10, 13, 22, 28,
                                       18, 15, 23, 31, 17, 16, 25, 24, 14, 2, 3, 1, 0, 5, 4, 42, 41, 43, 46, 47, 45, 48, 44, 50, 49};
  return dir == 1 ? u8 : dir == 2 ? adj : f32;
}

// Rows whose delays follow no pattern (DM lists or channels in descending order, shuffled
// or very uneven lists) cost a row-block variant its slots and the way there, 1.2
// times its time on regular lists, where the jump form takes 1.06 whatever the list
// (1024 channels, 2000 DM trials, 20,000 samples: 0.95 ms in row blocks, 1.12 with the DM
// list reversed, 1.01 slot by slot; backward, 1024 DM trials, channels in descending order:
// 0.80, 0.97 and 0.84).  So the jump form is kept for them.
int slots_variant(int vi) { return vi == 35 ? 49 : vi == 37 ? 50 : -1; }

// The choice by size.  A plan that was not tuned keeps, beside its default
// variant, a few with smaller tiles, and each call takes the one with the least
// estimated time,
//   max(start + rows * alone * f, rounds * (turn + rows * full * f)),   rounds = ceil(blocks / CUs),
//   f = 1 + chain * s, with weights also times `weights`,
// in us, rows the input rows, fitted to about 2000 random calls on MI355X: start and `alone` with at
// most one block per CU (the latency of a row's step), turn and `full` a block's share of a CU that holds as many as
// fit (turn: the tile's prologue and outputs, which with one block per CU nothing hides, and in the
// adjoint its partial sums); s is the share of rows without a pattern, `chain` what they cost.  The coarse tiles
// have the best throughput (64 DM trials x 1280 samples: 39 adds per ns over the chip; 16 x
// 256 in LDS: 17), the fine ones occupy the chip with little work: 1024 channels, 301 DM trials, 2003 samples are 10 coarse
// tiles in 473 us or 304 fine ones in 103 us, while 370 channels, 1072 DM trials,
// 11,790 samples are 170 coarse tiles in 193 us and 315 us in fine ones.  Tiles of
// 48 DM trials (3 waves per SIMD, 0.85 of the coarse tile's time) take the calls
// that would leave the last round of coarse tiles half empty, and tiles of 32 x
// 768 those between the sizes (two blocks per CU share one's waits: 2 beams of 264
// channels, 239 DM trials, 18,314 samples take 106 us, 132 us in coarse tiles and 153
// in LDS; backward 93, 125 and 170).  Beside the wide windows (39, 40: 8 to 12 samples between
// neighbouring rows) also 16 x 768 samples in a window of 48 (11) and, forward, 16 x 512 (46) are
// kept, whose blocks share a CU: 8 beams of 20 channels, 256 DM trials, 27,155 samples
// take 122 us in 39 and 86 in 11, while 3 of 592 channels, 605 DM trials, 15,894 samples take
// 663 and 1094.  The wide lane tiles (48) are kept where delay spans
// leave no other lane kernel (backward, 30 channels x 102 DM trials x 2162 samples: 18.5
// us, 61 in the default's wide windows), and the direct kernel, which stages nothing, takes
// the calls of a few rows (12 channels, 18 DM trials, 2793 samples backward: 6.7 us, 8.6),
// weighted also larger ones whose input an L2 holds (170 us, 241 in the wide lane tiles on 1294
// channels, 16 DM trials, 464 samples; past it 247 and 168 on 883 channels, 75, 1552).
// Weights cost the lane kernels, which apply them to each term, and a little the smaller row
// blocks the factor `weights` more than the others.  Over 150 random calls each way (1 to 40 beams, 8 to 1536 channels, 8
// to 3000 DM trials, 200 to 60,000 samples; profiles/choice_by_size.txt) the time is 2 to 3 %
// from the fastest kernel's on average (uint8 5 %), within 15 % in nine of ten, and 1.4 to 1.6 times at
// most, where the input rows are few or the gradient's rows shorter than the delays.
struct SizeCost {
  int vi;
  float start, alone, turn, full, chain, weights;
  enum { any_plan, wide_plan, if_default } kept = any_plan;  // beside which defaults it is kept
};
static constexpr int kWideLanes = 48;
static const std::vector<SizeCost>& size_costs(int dir) {
  constexpr auto wide = SizeCost::wide_plan;
  constexpr auto main = SizeCost::if_default;
  static const std::vector<SizeCost> f32 = {{35, 9.3f, .441f, 21.f, .478f, .25f, 1.f},
                                            {49, 9.8f, .460f, 21.f, .500f, 0.f, 1.f, main},
                                            {39, 7.9f, .414f, 17.f, .450f, 0.f, 1.f, main},
                                            {40, 5.4f, .509f, 5.0f, .220f, 0.f, 1.f, main},
                                            {41, 8.3f, .400f, 16.2f, .420f, .32f, 1.07f},
                                            {43, 5.0f, .286f, 5.3f, .181f, .45f, 1.08f},
                                            {44, 2.9f, .074f, 1.0f, .037f, 0.f, 1.36f},
                                            {45, 3.0f, .113f, 1.0f, .0625f, 0.f, 1.16f},
                                            {46, 3.1f, .163f, 1.5f, .126f, 0.f, 1.f, wide},
                                            {11, 3.3f, .347f, 1.7f, .150f, 0.f, 1.f, wide},
                                            {kWideLanes, 2.8f, .126f, 1.6f, .136f, 0.f, 1.24f}};
  // (two rounds of 23 are one of 22: on few channels they cost less, where the 8 us that do not
  // grow with the channels weigh most, on many more: 256 channels, 2048 DM trials, 60,000
  // samples take 0.735 ms in 22 and 0.761 in 23)
  static const std::vector<SizeCost> u8 = {{22, 5.5f, .456f, 8.0f, .357f, 0.f, 1.f},
                                           {23, 4.6f, .268f, 3.9f, .200f, 0.f, 1.f},
                                           {25, 3.7f, .180f, 2.2f, .122f, 0.f, 1.f},
                                           {26, 3.4f, .127f, 1.4f, .080f, 0.f, 1.f},
                                           {27, 3.6f, .132f, 2.1f, .138f, 0.f, 1.f}};
  static const std::vector<SizeCost> adj = {{37, 22.7f, .465f, 50.f, .485f, .2f, 1.f},
                                            {50, 22.9f, .489f, 50.f, .510f, 0.f, 1.f, main},
                                            {42, 19.6f, .425f, 33.f, .428f, .27f, 1.f},
                                            {39, 17.9f, .452f, 36.f, .470f, 0.f, 1.f},
                                            {40, 13.7f, .599f, 15.f, .215f, 0.f, 1.f, main},
                                            {43, 13.1f, .283f, 10.f, .190f, .42f, 1.f},
                                            {44, 6.1f, .0735f, 2.3f, .0355f, 0.f, 1.f},
                                            {46, 8.3f, .172f, 5.8f, .127f, 0.f, 1.f},
                                            {11, 9.7f, .400f, 9.2f, .130f, 0.f, 1.f, wide},
                                            {kWideLanes, 7.1f, .125f, 5.9f, .135f, 0.f, 1.f}};
  return dir == 1 ? u8 : dir == 2 ? adj : f32;
}

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

static float size_cost(dedisp_plan p, int dir, const Variant& v, int nbeam, int64_t nout, bool weighted) {
  // variants that were not measured (wide spans): the coarse tile's rate, scaled by the tile
  SizeCost c = {v.id, 2.f, .47f, 2.f, .508f * (float)(v.dt() * v.st()) / (64 * 1280), 0.f, 1.f};
  for (const SizeCost& k : size_costs(dir))
    if (k.vi == v.id) c = k;
  const int64_t rows_out = dir == 2 ? p->nchan : p->ndm, rows_in = dir == 2 ? p->ndm : p->nchan;
  const float rounds = (float)ceil_div(ceil_div(rows_out, v.dt()) * ceil_div(nout, v.st()) * nbeam, p->ncu);
  const auto plain = p->plain[dir].find(v.id);  // (known for every variant the choice can take)
  const float s = c.chain > 0.f && plain != p->plain[dir].end() ? plain->second : 0.f;
  const float rows = rows_in * (1.f + c.chain * s) * (weighted ? c.weights : 1.f);
  return std::max(c.start + rows * c.alone, rounds * (c.turn + rows * c.full));
}

// The direct kernel's (float32): a term's latency, forward longer where the input is
// more than an L2 holds, or with several blocks of 256 outputs per CU its share; the
// adjoint's partial sums beside it.
static float direct_cost(dedisp_plan p, int dir, int nbeam, int64_t nout) {
  const int64_t rows_out = dir == 2 ? p->nchan : p->ndm, rows_in = dir == 2 ? p->ndm : p->nchan;
  const float blocks = (float)(rows_out * ceil_div(nout, 256) * nbeam);
  const bool in_l2 = nbeam * (int64_t)p->nchan * (nout + p->max_delay) * 4 <= 6 << 20;
  return (dir == 2 ? 5.f : 0.f) + rows_in * std::max(dir == 2 ? .2f : in_l2 ? .17f : .27f, blocks / p->ncu * .05f);
}

// The variant a call of nbeam x nout output samples runs (-1: direct).
static int pick_variant(dedisp_plan p, int dir, int nbeam, int64_t nout, bool weighted = false) {
  const int main = dir == 0 ? p->var_f32 : dir == 1 ? p->var_u8 : p->var_adj;
  if (!p->by_size[dir] || main < 0) return main;
  const std::vector<Variant>& vs = dir == 1 ? variants_u8() : variants_f32();
  // from 16 blocks per CU on the int32 stores bind, and the packed sums of the
  // default uint8 shape are as fast as any (0.40 ms against 0.41 to 0.44 ms on 32
  // channels, 2048 DM trials, 200,000 samples)
  const Variant& mv = vs[main];
  if (dir == 1 && mv.mode == 1 && ceil_div(p->ndm, mv.dt()) * ceil_div(nout, mv.st()) * nbeam >= 16 * (int64_t)p->ncu)
    return main;
  int best = main;
  float least = size_cost(p, dir, mv, nbeam, nout, weighted);
  for (int vi : p->fine[dir]) {
    const float c = size_cost(p, dir, vs[vi], nbeam, nout, weighted);
    if (c < least) {
      least = c;
      best = vi;
    }
  }
  return dir != 1 && direct_cost(p, dir, nbeam, nout) < least ? -1 : best;
}

static bool aligned16(const void* ptr) { return ((uintptr_t)ptr & 15u) == 0; }

// The uint8 and adjoint kernels are chosen (and their tables built) on first
// use or by dedisp_plan_prepare; -2 marks "not chosen yet".
static void ensure_chosen(dedisp_plan p, int dir) {
  int& v = dir == 0 ? p->var_f32 : dir == 1 ? p->var_u8 : p->var_adj;
  if (v != -2) return;
  // the first of the preference order that fits (else the direct kernel), and
  // what the choice by size may take beside it
  const std::vector<int>& order = default_order(dir);
  const size_t top = std::min<size_t>(4, order.size());
  std::vector<int> ask(order.begin(), order.begin() + top);
  for (const SizeCost& c : size_costs(dir)) ask.push_back(c.vi);
  int first = -1;
  for (size_t n : {top, order.size()}) {  // the rest is checked only if none of those fits
    if (first >= 0 || check_fits(p, dir, n == top ? ask : order) != DEDISP_OK) break;
    for (size_t k = 0; k < n && first < 0; ++k)
      if (p->fits[dir][order[k]] == 0) first = order[k];
  }
  p->by_size[dir] = true;
  p->fine[dir].clear();
  const int blocks = first;  // the row blocks' variant, if it is one
  const int slots = dir == 1 ? -1 : slots_variant(first);
  if (slots >= 0 && p->plain[dir][first] > kSlotsShare && check_fits(p, dir, {slots}) == DEDISP_OK &&
      p->fits[dir][slots] == 0)
    first = slots;
  v = first;
  if (first < 0) return;
  std::vector<int> build = {first};
  const bool wide = first == 39 || first == 40;  // the wide windows
  bool lanes = false;                            // a lane kernel fits
  auto wanted = [&](const SizeCost& c) {
    if (c.vi == first || c.vi == blocks || c.vi == slots || c.kept == SizeCost::if_default ||
        (c.kept == SizeCost::wide_plan && !wide) || p->fits[dir][c.vi] != 0 || (c.vi == kWideLanes && lanes && dir != 1))
      return false;
    lanes |= dir != 1 && variants_f32()[c.vi].kind == KIND_LANE_F32;
    return true;
  };
  for (const SizeCost& c : size_costs(dir))
    if (wanted(c)) build.push_back(c.vi);
  const std::vector<int> all = build;
  std::map<int, Tables>& m = dir == 0 ? p->fwd_f32 : dir == 1 ? p->fwd_u8 : p->adj_f32;
  build.erase(std::remove_if(build.begin(), build.end(), [&](int vi) { return m.count(vi) != 0; }), build.end());
  if (build.empty() || build_tables(p, dir, build) == DEDISP_OK) {
    p->fine[dir].assign(all.begin() + 1, all.end());
  } else if (ensure_tables(p, dir, first, nullptr) != DEDISP_OK) {
    v = -1;
  }
}

// Scratch of the allocation-free adjoint (dedisp_adjoint_noalloc): the
// per-tile FP64 partial sums of the weight gradient.  Every GPU the library
// runs on holds its own copy until the process ends.  Host code never uses
// the array's name as an address: the device address of the current
// device's copy comes from scratch_address().
constexpr size_t kNoAllocScratchBytes = DEDISP_ADJOINT_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) double scratch[kNoAllocScratchBytes / sizeof(double)];

// Device address of the current device's scratch, looked up once per device
// (at plan creation, with that device current); nullptr with the error set
// if the lookup fails.
static void* scratch_address(int device) {
  static std::mutex mu;
  static std::map<int, void*> addr;
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find(device);
  if (it != addr.end()) return it->second;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    (void)hip_fail(e == hipSuccess ? hipErrorInvalidSymbol : e, "looking up the adjoint scratch array");
    return nullptr;
  }
  addr[device] = ptr;
  return ptr;
}

// FP64 partial sums of the weight gradient with variant vi: one per channel and
// (beam, time part), 256-sample parts for the direct kernel, the variant's time
// tiles otherwise.
static size_t partial_bytes(dedisp_plan p, int vi, int nbeam, int64_t nin) {
  const int64_t part = vi < 0 ? 256 : variants_f32()[vi].st();
  return (size_t)nbeam * (size_t)((nin + part - 1) / part) * (size_t)p->nchan * sizeof(double);
}

// The variant of an adjoint call: the choice by size, except where only the default
// variant's partial sums fit the fixed scratch (few channels and long rows take
// short tiles: 8 channels, 36e6 samples need 9.0 MB in tiles of 256 samples and 1.8 MB
// in those of 1280).  Calls with a workspace choose the same, so that both entry
// points give the same bits.
static int pick_adjoint(dedisp_plan p, int nbeam, int64_t nin, bool grad_w) {
  const int vi = pick_variant(p, 2, nbeam, nin);
  return grad_w && partial_bytes(p, vi, nbeam, nin) > kNoAllocScratchBytes &&
                 partial_bytes(p, p->var_adj, nbeam, nin) <= kNoAllocScratchBytes
             ? p->var_adj
             : vi;
}

// The adjoint's launches by variant vi with the partial-sum buffer given (null
// when no weight gradient is asked for).  With may_allocate false the
// variant's tables must exist already (nothing is built).
static dedisp_status adjoint_impl(dedisp_plan p, int vi, int32_t nbeam, int32_t nsamp, int32_t nin, const float* d_g,
                                  int64_t g_stride, const float* d_w, const float* d_in, int64_t in_stride,
                                  float* d_grad_in, int64_t gi_stride, float* d_grad_w, double* partial,
                                  hipStream_t s, bool may_allocate) {
  hipError_t e;
  int nparts;
  if (vi < 0) {
    e = launch_direct_adjoint(d_g, g_stride, g_stride * p->ndm, p->d_delay, p->nchan, p->ndm, nsamp, nin, d_w,
                              d_grad_in, gi_stride, gi_stride * p->nchan, d_in, in_stride, in_stride * p->nchan,
                              partial, nbeam, s);
    if (e != hipSuccess) return hip_fail(e, "launching the direct adjoint kernel");
    nparts = nbeam * ((nin + 255) / 256);
  } else {
    Tables* t = nullptr;
    if (may_allocate) {
      dedisp_status st = ensure_tables(p, 2, vi, &t);
      if (st != DEDISP_OK) return st;
    } else {
      auto it = p->adj_f32.find(vi);
      if (it == p->adj_f32.end())
        return fail(DEDISP_E_INVALID, "the adjoint tile tables are not built: call dedisp_plan_prepare first");
      t = &it->second;
    }
    const Variant& v = variants_f32()[vi];
    TileArgs a = {};
    a.in = d_g;
    a.in_stride = g_stride;
    a.in_beam_stride = g_stride * p->ndm;
    a.in_shift = -p->adj_pad;
    a.in_lo = p->adj_pad;
    a.in_hi = p->adj_pad + nsamp;
    a.rows_in = p->ndm;
    a.rows_out = p->nchan;
    a.nout = nin;
    a.n_time_tiles = (nin + v.st() - 1) / v.st();
    a.n_row_tiles = t->n_row_tiles;
    a.blk = t->d_blk;
    a.wav = t->d_wav;
    a.span = t->d_span;
    a.w_in = nullptr;
    a.out = d_grad_in;
    a.out_stride = gi_stride;
    a.out_beam_stride = gi_stride * p->nchan;
    a.w_out = d_w;
    a.x = d_in;
    a.x_stride = in_stride;
    a.x_beam_stride = in_stride * p->nchan;
    a.partial = partial;
    e = launch_tiled(v, a, nbeam, true, s);
    if (e != hipSuccess) return hip_fail(e, "launching the tiled adjoint kernel");
    nparts = nbeam * a.n_time_tiles;
  }
  if (d_grad_w) {
    e = launch_reduce_gradw(partial, nparts, p->nchan, d_grad_w, s);
    if (e != hipSuccess) return hip_fail(e, "launching the grad_w reduction");
  }
  return DEDISP_OK;
}

// Argument checks shared by both adjoint entry points.
static dedisp_status adjoint_check(dedisp_plan p, int32_t nbeam, int32_t nsamp, int32_t nin, const float* d_g,
                                   int64_t g_stride, const float* d_w, const float* d_in, int64_t in_stride,
                                   float* d_grad_in, int64_t gi_stride, float* d_grad_w) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (nbeam < 1 || nsamp < 1 || nin < 1) return fail(DEDISP_E_INVALID, "nbeam, nsamp and nin must be >= 1");
  if (nbeam > kMaxBeams) return fail(DEDISP_E_SHAPE, "at most 65535 beams per call");
  if (!d_g) return fail(DEDISP_E_INVALID, "output gradient is NULL");
  if (d_grad_w && !d_in) return fail(DEDISP_E_INVALID, "grad_w needs the forward input");
  if (g_stride < nsamp) return fail(DEDISP_E_SHAPE, "g_stride < nsamp");
  if (d_grad_in && gi_stride < nin) return fail(DEDISP_E_SHAPE, "gi_stride < nin");
  if (d_in && in_stride < nin) return fail(DEDISP_E_SHAPE, "in_stride < nin");
  if ((int64_t)nsamp + p->max_delay > nin) return fail(DEDISP_E_SHAPE, "nin < nsamp + max_delay");
  if (nin > kMaxRow || g_stride > kMaxRow || (d_in && in_stride > kMaxRow) || (d_grad_in && gi_stride > kMaxRow))
    return fail(DEDISP_E_SHAPE, "rows longer than 2^29 samples are not supported");
  if (!aligned16(d_g) || (g_stride * 4) % 16 || (d_grad_in && (!aligned16(d_grad_in) || (gi_stride * 4) % 16)) ||
      (d_in && (!aligned16(d_in) || (in_stride * 4) % 16)) || (d_w && ((uintptr_t)d_w & 3)))
    return fail(DEDISP_E_ALIGN, "pointers and row byte sizes must be multiples of 16 bytes");
  return DEDISP_OK;
}

}  // namespace dd

using namespace dd;

extern "C" {

const char* dedisp_status_string(dedisp_status s) {
  switch (s) {
    case DEDISP_OK: return "ok";
    case DEDISP_E_INVALID: return "invalid argument";
    case DEDISP_E_SHAPE: return "invalid shape or stride";
    case DEDISP_E_DTYPE: return "unsupported data type";
    case DEDISP_E_ALIGN: return "misaligned pointer or row";
    case DEDISP_E_NOMEM: return "out of memory";
    case DEDISP_E_HIP: return "HIP runtime error";
    case DEDISP_E_UNTUNED: return "no kernel variant fits";
    case DEDISP_E_WORKSPACE: return "workspace too small";
  }
  return "unknown status";
}

const char* dedisp_last_error(void) { return g_last_error.c_str(); }

dedisp_status dedisp_plan_create(dedisp_plan* plan, int32_t nchan, const double* freq_mhz, double tsamp_s,
                                 int32_t ndm, const double* dm) {
  if (!plan) return fail(DEDISP_E_INVALID, "plan pointer is NULL");
  *plan = nullptr;
  if (nchan < 1 || ndm < 1) return fail(DEDISP_E_INVALID, "nchan and ndm must be >= 1");
  if (!freq_mhz || !dm) return fail(DEDISP_E_INVALID, "frequency or DM array is NULL");
  if (!(tsamp_s > 0.0) || !std::isfinite(tsamp_s)) return fail(DEDISP_E_INVALID, "tsamp must be > 0 and finite");
  dedisp_plan p = new (std::nothrow) dedisp_plan_s();
  if (!p) return fail(DEDISP_E_NOMEM, "host allocation failed");
  p->nchan = nchan;
  p->ndm = ndm;
  p->tsamp = tsamp_s;
  p->freq.assign(freq_mhz, freq_mhz + nchan);
  p->dm.assign(dm, dm + ndm);
  dedisp_status st = build_delay_table(nchan, freq_mhz, tsamp_s, ndm, dm, p->delay, p->max_delay);
  if (st != DEDISP_OK) {
    delete p;
    return st;
  }
  p->adj_pad = (p->max_delay + 3) & ~3;
  hipError_t e = hipGetDevice(&p->device);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&p->ncu, hipDeviceAttributeMultiprocessorCount, p->device);
  if (e == hipSuccess && p->ncu < 1) p->ncu = 1;
  if (e == hipSuccess) e = hipMalloc(&p->d_delay, (p->delay.size() + 2 * kFitBatch) * sizeof(int32_t));
  if (e == hipSuccess)
    e = hipMemcpy(p->d_delay, p->delay.data(), p->delay.size() * sizeof(int32_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    st = hip_fail(e, "uploading the delay table");
    dedisp_plan_destroy(p);
    return st;
  }
  p->d_bad = p->d_delay + p->delay.size();
  // the allocation-free adjoint's scratch on this device, looked up once
  if (!scratch_address(p->device)) {
    st = DEDISP_E_HIP;
    dedisp_plan_destroy(p);
    return st;
  }
  ensure_chosen(p, 0);
  *plan = p;
  return DEDISP_OK;
}

dedisp_status dedisp_compute_delays(int32_t nchan, const double* freq_mhz, double tsamp_s, int32_t ndm,
                                    const double* dm, int32_t* host, int32_t* max_delay) {
  if (nchan < 1 || ndm < 1) return fail(DEDISP_E_INVALID, "nchan and ndm must be >= 1");
  if (!freq_mhz || !dm || !host) return fail(DEDISP_E_INVALID, "an array pointer is NULL");
  if (!(tsamp_s > 0.0) || !std::isfinite(tsamp_s)) return fail(DEDISP_E_INVALID, "tsamp must be > 0 and finite");
  std::vector<int32_t> t;
  int md = 0;
  dedisp_status st = build_delay_table(nchan, freq_mhz, tsamp_s, ndm, dm, t, md);
  if (st != DEDISP_OK) return st;
  memcpy(host, t.data(), t.size() * sizeof(int32_t));
  if (max_delay) *max_delay = md;
  return DEDISP_OK;
}

dedisp_status dedisp_plan_destroy(dedisp_plan p) {
  if (!p) return DEDISP_OK;
  if (p->d_delay) (void)hipFree(p->d_delay);
  delete p;
  return DEDISP_OK;
}

dedisp_status dedisp_plan_info(dedisp_plan p, int32_t* nchan, int32_t* ndm, int32_t* max_delay) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (nchan) *nchan = p->nchan;
  if (ndm) *ndm = p->ndm;
  if (max_delay) *max_delay = p->max_delay;
  return DEDISP_OK;
}

dedisp_status dedisp_plan_delays(dedisp_plan p, int32_t* host) {
  if (!p || !host) return fail(DEDISP_E_INVALID, "plan or output is NULL");
  memcpy(host, p->delay.data(), p->delay.size() * sizeof(int32_t));
  return DEDISP_OK;
}

int32_t dedisp_variant_count(dedisp_dtype t) {
  return t == DEDISP_U8 ? (int32_t)variants_u8().size() : t == DEDISP_F32 ? (int32_t)variants_f32().size() : 0;
}

const char* dedisp_variant_name(dedisp_dtype t, int32_t i) {
  if (t == DEDISP_U8 && i >= 0 && i < (int)variants_u8().size()) return variants_u8()[i].name;
  if (t == DEDISP_F32 && i >= 0 && i < (int)variants_f32().size()) return variants_f32()[i].name;
  return nullptr;
}

dedisp_status dedisp_plan_set_variant(dedisp_plan p, dedisp_dtype t, int32_t vi) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (t != DEDISP_F32 && t != DEDISP_U8) return fail(DEDISP_E_DTYPE, "dtype must be F32 or U8");
  const int dir = t == DEDISP_U8 ? 1 : 0;
  if (vi >= 0) {
    dedisp_status st = ensure_tables(p, dir, vi, nullptr);
    if (st != DEDISP_OK) return st;
  } else if (vi != -1) {
    return fail(DEDISP_E_INVALID, "variant must be >= -1");
  }
  (t == DEDISP_U8 ? p->var_u8 : p->var_f32) = vi;
  p->by_size[dir] = false;
  return DEDISP_OK;
}

int32_t dedisp_plan_variant(dedisp_plan p, dedisp_dtype t) {
  if (!p) return -2;
  ensure_chosen(p, t == DEDISP_U8 ? 1 : 0);
  return t == DEDISP_U8 ? p->var_u8 : p->var_f32;
}

dedisp_status dedisp_plan_set_adjoint_variant(dedisp_plan p, int32_t vi) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (vi >= 0) {
    dedisp_status st = ensure_tables(p, 2, vi, nullptr);
    if (st != DEDISP_OK) return st;
  } else if (vi != -1) {
    return fail(DEDISP_E_INVALID, "variant must be >= -1");
  }
  p->var_adj = vi;
  p->by_size[2] = false;
  return DEDISP_OK;
}

int32_t dedisp_plan_adjoint_variant(dedisp_plan p) {
  if (!p) return -2;
  ensure_chosen(p, 2);
  return p->var_adj;
}

dedisp_status dedisp_plan_prepare(dedisp_plan p, dedisp_dtype t, int32_t adjoint) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (t != DEDISP_F32 && t != DEDISP_U8) return fail(DEDISP_E_DTYPE, "dtype must be F32 or U8");
  if (adjoint && t != DEDISP_F32) return fail(DEDISP_E_DTYPE, "the adjoint is float32 only");
  const int dir = adjoint ? 2 : (t == DEDISP_U8 ? 1 : 0);
  ensure_chosen(p, dir);
  const int v = dir == 0 ? p->var_f32 : dir == 1 ? p->var_u8 : p->var_adj;
  return v < 0 ? DEDISP_OK : ensure_tables(p, dir, v, nullptr);
}

dedisp_status dedisp_execute(dedisp_plan p, int32_t nbeam, int32_t nsamp, const void* d_in, dedisp_dtype in_type,
                             int64_t in_stride, const float* d_w, void* d_out, dedisp_dtype out_type,
                             int64_t out_stride, void* stream) {
  if (!p) return fail(DEDISP_E_INVALID, "plan is NULL");
  if (nbeam < 1 || nsamp < 1) return fail(DEDISP_E_INVALID, "nbeam and nsamp must be >= 1");
  if (nbeam > kMaxBeams) return fail(DEDISP_E_SHAPE, "at most 65535 beams per call");
  if (!d_in || !d_out) return fail(DEDISP_E_INVALID, "input or output pointer is NULL");
  const bool f32 = in_type == DEDISP_F32 && out_type == DEDISP_F32;
  const bool u8 = in_type == DEDISP_U8 && out_type == DEDISP_I32;
  if (!f32 && !u8) return fail(DEDISP_E_DTYPE, "supported pairs: F32->F32, U8->I32");
  if (u8 && d_w) return fail(DEDISP_E_DTYPE, "weights are not supported for uint8 input");
  if (in_stride < (int64_t)nsamp + p->max_delay) return fail(DEDISP_E_SHAPE, "in_stride < nsamp + max_delay");
  if (out_stride < nsamp) return fail(DEDISP_E_SHAPE, "out_stride < nsamp");
  if (in_stride > kMaxRow || (int64_t)nsamp + p->max_delay > kMaxRow)
    return fail(DEDISP_E_SHAPE, "rows longer than 2^29 samples are not supported");
  const int esz = u8 ? 1 : 4;
  if (!aligned16(d_in) || !aligned16(d_out) || (in_stride * esz) % 16 || (out_stride * 4) % 16 ||
      (d_w && ((uintptr_t)d_w & 3)))
    return fail(DEDISP_E_ALIGN, "pointers and row byte sizes must be multiples of 16 bytes");
  hipStream_t s = (hipStream_t)stream;
  ensure_chosen(p, u8 ? 1 : 0);
  const int vi = pick_variant(p, u8 ? 1 : 0, nbeam, nsamp, d_w != nullptr);
  hipError_t e;
  if (vi < 0) {
    if (u8)
      e = launch_direct_u8((const uint8_t*)d_in, in_stride, in_stride * p->nchan, p->d_delay, p->nchan, p->ndm,
                           (int32_t*)d_out, out_stride, out_stride * p->ndm, nsamp, nbeam, s);
    else
      e = launch_direct_f32((const float*)d_in, in_stride, in_stride * p->nchan, p->d_delay, p->nchan, p->ndm, d_w,
                            (float*)d_out, out_stride, out_stride * p->ndm, nsamp, nbeam, s);
    return e == hipSuccess ? DEDISP_OK : hip_fail(e, "launching the direct kernel");
  }
  const int dir = u8 ? 1 : 0;
  Tables* t = nullptr;
  dedisp_status st = ensure_tables(p, dir, vi, &t);
  if (st != DEDISP_OK) return st;
  const Variant& v = (u8 ? variants_u8() : variants_f32())[vi];
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
  a.n_time_tiles = (nsamp + v.st() - 1) / v.st();
  a.n_row_tiles = t->n_row_tiles;
  // blocks that walk several time tiles: about six per CU in total
  a.tiles_per_block = (int)std::max<int64_t>(
      1, std::min<int64_t>(a.n_time_tiles, (int64_t)a.n_time_tiles * a.n_row_tiles * nbeam / (6 * p->ncu)));
  a.blk = t->d_blk;
  a.wav = t->d_wav;
  a.w_in = d_w;
  a.out = d_out;
  a.out_stride = out_stride;
  a.out_beam_stride = out_stride * p->ndm;
  e = launch_tiled(v, a, nbeam, false, s);
  return e == hipSuccess ? DEDISP_OK : hip_fail(e, "launching the tiled kernel");
}

size_t dedisp_adjoint_workspace_bytes(dedisp_plan p, int32_t nbeam, int32_t nin) {
  if (!p || nbeam < 1 || nin < 1) return 0;
  // Enough for the direct kernel (256-sample parts) and every tiled variant.
  const int64_t parts = (int64_t)nbeam * ((nin + 255) / 256);
  return (size_t)parts * p->nchan * sizeof(double);
}

dedisp_status dedisp_adjoint(dedisp_plan p, int32_t nbeam, int32_t nsamp, int32_t nin, const float* d_g,
                             int64_t g_stride, const float* d_w, const float* d_in, int64_t in_stride,
                             float* d_grad_in, int64_t gi_stride, float* d_grad_w, void* d_ws, size_t ws_bytes,
                             void* stream) {
  dedisp_status st =
      adjoint_check(p, nbeam, nsamp, nin, d_g, g_stride, d_w, d_in, in_stride, d_grad_in, gi_stride, d_grad_w);
  if (st != DEDISP_OK) return st;
  if (!d_grad_in && !d_grad_w) return DEDISP_OK;
  if (d_grad_w) {
    if (!d_ws) return fail(DEDISP_E_WORKSPACE, "workspace is NULL");
    if (ws_bytes < dedisp_adjoint_workspace_bytes(p, nbeam, nin)) return fail(DEDISP_E_WORKSPACE, "workspace too small");
    if ((uintptr_t)d_ws & 7) return fail(DEDISP_E_ALIGN, "workspace must be 8-byte aligned");
  }
  ensure_chosen(p, 2);
  return adjoint_impl(p, pick_adjoint(p, nbeam, nin, d_grad_w != nullptr), nbeam, nsamp, nin, d_g, g_stride, d_w, d_in,
                      in_stride, d_grad_in, gi_stride, d_grad_w, d_grad_w ? (double*)d_ws : nullptr, (hipStream_t)stream,
                      true);
}

size_t dedisp_adjoint_noalloc_bytes(dedisp_plan p, int32_t nbeam, int32_t nin) {
  if (!p || nbeam < 1 || nin < 1 || p->var_adj == -2) return 0;
  return partial_bytes(p, pick_adjoint(p, nbeam, nin, true), nbeam, nin);
}

dedisp_status dedisp_adjoint_noalloc(dedisp_plan p, int32_t nbeam, int32_t nsamp, int32_t nin, const float* d_g,
                                     int64_t g_stride, const float* d_w, const float* d_in, int64_t in_stride,
                                     float* d_grad_in, int64_t gi_stride, float* d_grad_w, void* stream) {
  dedisp_status st =
      adjoint_check(p, nbeam, nsamp, nin, d_g, g_stride, d_w, d_in, in_stride, d_grad_in, gi_stride, d_grad_w);
  if (st != DEDISP_OK) return st;
  if (!d_grad_in && !d_grad_w) return DEDISP_OK;
  if (p->var_adj == -2)
    return fail(DEDISP_E_INVALID, "the adjoint kernel is not chosen yet: call dedisp_plan_prepare first");
  double* partial = nullptr;
  if (d_grad_w) {
    const size_t need = dedisp_adjoint_noalloc_bytes(p, nbeam, nin);
    if (need > kNoAllocScratchBytes)
      return fail(DEDISP_E_WORKSPACE, "the weight gradient's partial sums (" + std::to_string(need) +
                                          " bytes) exceed the fixed scratch of " +
                                          std::to_string(kNoAllocScratchBytes) + " bytes; use dedisp_adjoint");
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "querying the current device");
    if (dev != p->device) return fail(DEDISP_E_INVALID, "the plan belongs to another device");
    partial = static_cast<double*>(scratch_address(dev));
    if (!partial) return DEDISP_E_HIP;
  }
  return adjoint_impl(p, pick_adjoint(p, nbeam, nin, d_grad_w != nullptr), nbeam, nsamp, nin, d_g, g_stride, d_w, d_in,
                      in_stride, d_grad_in, gi_stride, d_grad_w, partial, (hipStream_t)stream, false);
}

}  // extern "C"
