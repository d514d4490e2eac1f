// gfx950 kernels for brute-force incoherent dedispersion.
//
// Forward map (Sclocco et al., arXiv 1601.01165, Section 2.1, Algorithm 1):
//   out[b][r][t] = sum over input rows c, ascending, of w[c] * in[b][c][t + delta(r, c)]
// with r a DM trial and c a channel.  The adjoint is the same map with the
// roles swapped (r a channel, c a DM trial, delay' = pad - delay, input rows
// read as zero outside the output range), so one tile engine serves both.
//
// Parallel structure (Section 2.2): each work item owns (output row, time)
// pairs; a block owns a tile of output rows x time samples, so the input rows
// it needs are shared by all its rows (the paper's DM-direction reuse through
// local memory).  On gfx950:
//   * a block stages, for cc input rows at a time, the window
//     [t0 + stage_base(c), t0 + stage_base(c) + stage_len(c)) of each row into
//     LDS with 16-byte loads (all 16-byte aligned);
//   * each wave owns dpw output rows and 64*tp samples, each lane tp
//     consecutive samples.  Per input row the lane copies its window of
//     samples from LDS into registers once (16-byte LDS reads) and every one
//     of its dpw rows adds the tp window registers that start at the row's
//     delay offset, selected by jumping into static code: a block per row for
//     regular DM lists, one per output row, or through VGPR index mode (see
//     gen_win_asm.py).  One LDS byte
//     thus feeds several adds, which is what keeps the add units busy: an LDS
//     read per add would cap the rate at the LDS bandwidth.
//   * blocks are remapped so that the blocks of one time tile run on the same
//     XCD, sharing that XCD's L2 for the input window.
//   * accumulation order per output is ascending input row with one rounding
//     per term, the order of Algorithm 1, so the FP32 results are those of a
//     sequential FP32 loop.
#pragma once

#include "detect_dev.h"
#include "device_util.h"
#include "internal.h"

namespace dd {

typedef float v16f __attribute__((ext_vector_type(16)));
#include "win_asm.inc"

// ---------------------------------------------------------------------------
// FP32 tile engine with the register window.
// ---------------------------------------------------------------------------

// Stage input rows [c0, c0 + ncc) into LDS.  Wave w copies rows w, w + NWAVE, ...
// With weights each staged sample is the FP32 product w[c] * x (the weight is
// a gain on the channel's data), so the sums themselves are plain adds.
template <int NWAVE, int ROWCAP, bool WEIGHTED>
__device__ __forceinline__ void stage_f32(int wave, float4* lds4, const float* in, const TileArgs& a, const int32_t* blk,
                                          int c0, int ncc, int t0) {
  const int lane = lane_fresh();
  for (int cl = wave; cl < ncc; cl += NWAVE) {
    const int sb = blk[2 * (c0 + cl)];
    const int sl = blk[2 * (c0 + cl) + 1];
    const float wc = WEIGHTED ? a.w_in[c0 + cl] : 1.f;
    const float* src = in + (int64_t)(c0 + cl) * a.in_stride + a.in_shift;
    const int u0 = t0 + sb;
    float4* dst = lds4 + cl * (ROWCAP / 4);
    const int nv = sl >> 2;
#pragma unroll 4
    for (int v = lane; v < nv; v += 64) {
      const int u = u0 + 4 * v;
      float4 x;
      if (u >= a.in_lo && u + 4 <= a.in_hi) {
        x = *reinterpret_cast<const float4*>(src + u);
      } else {
        x.x = (u + 0 >= a.in_lo && u + 0 < a.in_hi) ? src[u + 0] : 0.f;
        x.y = (u + 1 >= a.in_lo && u + 1 < a.in_hi) ? src[u + 1] : 0.f;
        x.z = (u + 2 >= a.in_lo && u + 2 < a.in_hi) ? src[u + 2] : 0.f;
        x.w = (u + 3 >= a.in_lo && u + 3 < a.in_hi) ? src[u + 3] : 0.f;
      }
      if (WEIGHTED) {
        x.x = wc * x.x;
        x.y = wc * x.y;
        x.z = wc * x.z;
        x.w = wc * x.w;
      }
      dst[v] = x;
    }
  }
}

// Asynchronous form: 16-byte buffer loads that write LDS directly (no VGPR
// round trip), completed by `s_waitcnt vmcnt(0)`.  Each row gets a buffer
// resource covering its valid range, so positions outside it read as zero
// without a branch (the adjoint relies on this for its virtual padding).
template <int NWAVE, int ROWCAP>
__device__ __forceinline__ void stage_f32_async(int wave, float4* lds4, const float* in, const TileArgs& a,
                                                const int32_t* blk, int c0, int ncc, int t0) {
  // whole 64-lane loads stay inside the row's LDS slot
  static_assert(ROWCAP % 256 == 0, "LDS rows hold a multiple of 64 float4");
  const int lane = lane_fresh();
  for (int cl = wave; cl < ncc; cl += NWAVE) {
    const ent2_t bl = sload_entry2(blk + 2 * (c0 + cl));
    const int sb = bl[0];
    const int sl = bl[1];
    const float* base = in + (int64_t)(c0 + cl) * a.in_stride + a.in_lo + a.in_shift;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (a.in_hi - a.in_lo) * 4, 0x00020000);
    const int u0 = t0 + sb - a.in_lo;
    const int nv = sl >> 2;
    for (int v0 = 0; v0 < nv; v0 += 64) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LDS_AS void*)(lds4 + cl * (ROWCAP / 4) + v0), 16,
                                               (u0 + 4 * (v0 + lane)) * 4, 0, 0, 0);
    }
  }
}

// Entries {stage base, stage length} of the rows wave w stages for the pass
// starting at input row c0 (rows w, w + NWAVE, ...): lane 2k holds the base
// of the wave's k-th row, lane 2k + 1 its length and lane 32 + k its weight
// (float bits; weighted kernels only).  A vector load, issued a pass ahead:
// the per-pass wait for the staged rows covers it, so staging never stalls on
// a scalar-cache miss.
template <int NWAVE, int CC>
__device__ __forceinline__ int32_t stage_entries(int wave, const int32_t* blk, const float* w, int rows_in, int c0) {
  constexpr int RPW = (CC + NWAVE - 1) / NWAVE;
  static_assert(2 * RPW <= 32, "entries and weights share one VGPR");
  const int lane = lane_fresh();
  if (lane < 32) {
    const int cl = wave + (lane >> 1) * NWAVE;
    if (lane < 2 * RPW && cl < CC && c0 + cl < rows_in) return blk[2 * (c0 + cl) + (lane & 1)];
  } else if (w) {
    const int cl = wave + (lane - 32) * NWAVE;
    if (lane - 32 < RPW && cl < CC && c0 + cl < rows_in) return __float_as_int(w[c0 + cl]);
  }
  return 0;
}

// Weighted kernels, asynchronous staging: once this wave's rows of a pass
// have landed, scale them in place by their channel's weight (FP32 product,
// the weight being a gain on the data), before the barrier that publishes the
// pass.  `ent` holds the pass's entries and weights (stage_entries).
template <int NWAVE, int ROWCAP>
__device__ __forceinline__ void scale_rows(int wave, float4* lds4, int32_t ent, int ncc) {
  for (int k = 0, cl = wave; cl < ncc; ++k, cl += NWAVE) {
    const int lane = lane_fresh();
    const int sl = __builtin_amdgcn_readlane(ent, 2 * k + 1);
    const float wc = __int_as_float(__builtin_amdgcn_readlane(ent, 32 + k));
    float4* row = lds4 + cl * (ROWCAP / 4);
    for (int v = lane; v < (sl >> 2); v += 64) {
      float4 x = row[v];
      x.x = wc * x.x;
      x.y = wc * x.y;
      x.z = wc * x.z;
      x.w = wc * x.w;
      row[v] = x;
    }
  }
}

// stage_f32_async with the entries from stage_entries (no scalar loads).
template <int NWAVE, int ROWCAP>
__device__ __forceinline__ void stage_f32_async_pre(int wave, float4* lds4, const float* in, const TileArgs& a, int32_t ent,
                                                    int c0, int ncc, int t0) {
  static_assert(ROWCAP % 256 == 0, "LDS rows hold a multiple of 64 float4");
  for (int k = 0, cl = wave; cl < ncc; ++k, cl += NWAVE) {
    const int lane = lane_fresh();
    const int sb = __builtin_amdgcn_readlane(ent, 2 * k);
    const int sl = __builtin_amdgcn_readlane(ent, 2 * k + 1);
    const float* base = in + (int64_t)(c0 + cl) * a.in_stride + a.in_lo + a.in_shift;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (a.in_hi - a.in_lo) * 4, 0x00020000);
    const int u0 = t0 + sb - a.in_lo;
    const int nv = sl >> 2;
    for (int v0 = 0; v0 < nv; v0 += 64) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LDS_AS void*)(lds4 + cl * (ROWCAP / 4) + v0), 16,
                                               (u0 + 4 * (v0 + lane)) * 4, 0, 0, 0);
    }
  }
}

// After the asynchronous loads of a pass have landed: rewrite the one 16-byte
// chunk per row that straddles the end of the valid range (valid elements
// from memory, the rest zero).  The loads check the range per 4 bytes and leave
// zeros there themselves (the lane kernels rely on it; tested with NaN in the rows'
// padding); this keeps the window kernels right without it.  Only the adjoint's
// range can end off a 16-byte boundary.
template <int NWAVE, int ROWCAP>
__device__ __forceinline__ void fix_tail_async(int wave, float4* lds4, const float* in, const TileArgs& a,
                                               const int32_t* blk, int c0, int ncc, int t0) {
  if ((a.in_hi & 3) == 0) return;
  const int lane = lane_fresh();
  const int hi4 = a.in_hi & ~3;
  for (int cl = wave; cl < ncc; cl += NWAVE) {
    const ent2_t bl = sload_entry2(blk + 2 * (c0 + cl));
    const int v = (hi4 - (t0 + bl[0])) >> 2;
    if (lane == 0 && v >= 0 && 4 * v < bl[1]) {
      const float* src = in + (int64_t)(c0 + cl) * a.in_stride + a.in_shift;
      float4 x;
      x.x = src[hi4];
      x.y = (hi4 + 1 < a.in_hi) ? src[hi4 + 1] : 0.f;
      x.z = (hi4 + 2 < a.in_hi) ? src[hi4 + 2] : 0.f;
      x.w = 0.f;
      lds4[cl * (ROWCAP / 4) + v] = x;
    }
  }
}

// Store a finished tile (adjoint: scaled by w_out, with the wave's partial
// sums of x * G for the weight gradient).
template <int TP, int DPW, int NWAVE, bool ADJ>
__device__ __forceinline__ void win_store(int wave, const TileArgs& a, const v16f* acc, int tt, int rt, int beam) {
  constexpr int DT = NWAVE * DPW;
  const int t0 = tt * 64 * TP;
  const int lane = lane_fresh();
  float* out = static_cast<float*>(a.out);
  const int tl = t0 + lane * TP;
#pragma unroll
  for (int jj = 0; jj < DPW; ++jj) {
    const int r = rt * DT + wave * DPW + jj;
    if (r >= a.rows_out) break;
    const float scale = (ADJ && a.w_out) ? a.w_out[r] : 1.f;
    double gw = 0.0;
    const float* xrow = nullptr;
    if (ADJ && a.partial) xrow = a.x + (int64_t)beam * a.x_beam_stride + (int64_t)r * a.x_stride;
    float* orow = out ? out + (int64_t)beam * a.out_beam_stride + (int64_t)r * a.out_stride : nullptr;
#pragma unroll
    for (int i4 = 0; i4 < TP / 4; ++i4) {
      const int e0 = jj * TP + 4 * i4;
      float4 v;
      v.x = acc[(e0 + 0) / 16][(e0 + 0) % 16];
      v.y = acc[(e0 + 1) / 16][(e0 + 1) % 16];
      v.z = acc[(e0 + 2) / 16][(e0 + 2) % 16];
      v.w = acc[(e0 + 3) / 16][(e0 + 3) % 16];
      const int t = tl + 4 * i4;
      if (ADJ && xrow) {
        if (t + 4 <= a.nout) {
          const float4 xv = *reinterpret_cast<const float4*>(xrow + t);
          gw += (double)xv.x * (double)v.x;
          gw += (double)xv.y * (double)v.y;
          gw += (double)xv.z * (double)v.z;
          gw += (double)xv.w * (double)v.w;
        } else {
          if (t + 0 < a.nout) gw += (double)xrow[t + 0] * (double)v.x;
          if (t + 1 < a.nout) gw += (double)xrow[t + 1] * (double)v.y;
          if (t + 2 < a.nout) gw += (double)xrow[t + 2] * (double)v.z;
          if (t + 3 < a.nout) gw += (double)xrow[t + 3] * (double)v.w;
        }
      }
      if (orow) {
        if (ADJ) {
          v.x *= scale;
          v.y *= scale;
          v.z *= scale;
          v.w *= scale;
        }
        if (t + 4 <= a.nout) {
          *reinterpret_cast<float4*>(orow + t) = v;
        } else {
          if (t + 0 < a.nout) orow[t + 0] = v.x;
          if (t + 1 < a.nout) orow[t + 1] = v.y;
          if (t + 2 < a.nout) orow[t + 2] = v.z;
          if (t + 3 < a.nout) orow[t + 3] = v.w;
        }
      }
    }
    if (ADJ && xrow) {
      // Fixed-order reduction over the 64 lanes of the wave.
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) gw += __shfl_xor(gw, m, 64);
      if (lane == 0) a.partial[((size_t)beam * a.n_time_tiles + tt) * a.rows_out + r] = gw;
    }
  }
}


// Single-pulse search in place of the store: each lane's TP consecutive
// samples of a row are its run of window starts; the look-ahead comes from
// the lanes above (DPP), so the rows never leave the registers.  Samples past
// the series end read as -inf.
template <int TP, int DPW, int NWAVE>
__device__ __forceinline__ void det_store_f32(int wave, const TileArgs& a, const v16f* acc, int tt, int rt, int beam, int t0) {
  constexpr int ST = 64 * TP;
  constexpr int DT = NWAVE * DPW;
  const int lane = lane_fresh();
  const int nvalid = min(ST, a.det_nsamp - t0);
  const int pos0 = TP * lane;
  const bool owned = pos0 < a.tile_step;
  const int lim = nvalid - pos0;
#pragma unroll
  for (int jj = 0; jj < DPW; ++jj) {
    const int r = rt * DT + wave * DPW + jj;
    if (r >= a.rows_out) break;
    float v[TP + kDetLook];
#pragma unroll
    for (int i = 0; i < TP; ++i) v[i] = acc[(jj * TP + i) / 16][(jj * TP + i) % 16];
    float bval[kDetNW];
    int bidx[kDetNW];
    double s1, s2;
    if (nvalid < ST) {
#pragma unroll
      for (int i = 0; i < TP; ++i) v[i] = i < lim ? v[i] : -INFINITY;
      det_lane_f32<TP, true>(v, owned, lim, bval, bidx, s1, s2);
    } else {
      det_lane_f32<TP, false>(v, owned, lim, bval, bidx, s1, s2);
    }
    det_commit_f32(a.det + ((int64_t)beam * a.rows_out + r) * a.n_time_tiles + tt, bval, bidx, s1, s2, pos0, t0);
  }
}

// NBUF = 1: synchronous staging through registers, one LDS buffer.
// NBUF = 2: asynchronous LDS loads into two buffers; the rows of pass p + 1
// are in flight while pass p is summed.
template <int TP, int DPW, int NWAVE, int NWIN, int CC, int ROWCAP, int NBUF, bool WEIGHTED, bool ADJ,
          bool DET = false, int JMP = 0>
__device__ __forceinline__ void win_tile(int wave, const TileArgs& a, int tt, int rt, int beam, float4* lds4) {
  constexpr int ST = 64 * TP;
  constexpr int DT = NWAVE * DPW;
  constexpr int NACC = TP * DPW / 16;
  constexpr bool RB = JMP == 3;  // one block of code per row
  static_assert(!RB || has_row_pass(TP, DPW, NWIN, JmpAcc0<TP, DPW, NWIN, CC>::value), "no row blocks for this shape");
  static_assert(Variant::kRowStub == kGenRowStub && Variant::row_block_bytes(TP, NWIN) == gen_row_block(TP, NWIN),
                "the tables' block offsets are not the generated code's");
  constexpr int WI = RB ? 4 : EntT<DPW>::ints;
  tt = __builtin_amdgcn_readfirstlane(tt);
  rt = __builtin_amdgcn_readfirstlane(rt);
  const int t0 = DET ? tt * a.tile_step : tt * ST;
  const int wt = rt * NWAVE + wave;
  const float* in = static_cast<const float*>(a.in) + (int64_t)beam * a.in_beam_stride;
  const int32_t* __restrict__ blk = uniform_ptr(a.blk + (size_t)rt * a.rows_in * 2);
  const int32_t* __restrict__ wav = uniform_ptr(a.wav + (size_t)wt * a.rows_in * WI);
  const float* w_in = WEIGHTED ? a.w_in : nullptr;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(LDS_AS float4*)(lds4);

  v16f acc[NACC];
#pragma unroll
  for (int q = 0; q < NACC; ++q) acc[q] = (v16f)(0.f);

  // The wave's table entry of the current input row lives in SGPRs; each
  // step fetches the next row's through a buffer resource (reads past the
  // last row return zero), advancing the byte offset itself.  Weights were
  // applied when the rows were staged, so the steps only add.
  typedef typename std::conditional<RB, ent4_t, typename EntT<DPW>::type>::type E;
  const __amdgpu_buffer_rsrc_t trs =
      __builtin_amdgcn_make_buffer_rsrc((void*)wav, (short)0, a.rows_in * WI * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(nullptr, (short)0, 0, 0x00020000);
  // the prefetching jump form holds two entries, the others load one ahead
  constexpr bool PF = JMP == 1 && DPW == 4;
  uint32_t toff = (PF ? 2 : 1) * WI * 4, woff = 4;
  E ea = sload_entry_t<E>(wav), eb;
  if (PF) eb = sbload_t<E>(trs, WI * 4);
  float wa = 0.f, wb = 0.f;
  const int npass = (a.rows_in + CC - 1) / CC;
  int32_t stg = 0;      // staging entries (and weights) of the next pass (NBUF = 2)
  int32_t stg_cur = 0;  // those of the pass being summed (weighted kernels)
  // Adjoint: the input rows (DM trials) of the passes at either end may stage
  // windows that all miss the valid samples [in_lo, in_hi) of the output
  // gradient (only zeros would be added); the tile runs from its first to
  // its last pass that meets them (all passes when no span table is given).
  int p_lo = 0, p_hi = npass - 1;
  if constexpr (ADJ) {
    if (a.span) {
      const int32_t* sp = uniform_ptr(a.span + (size_t)rt * npass * 2);
      auto live = [&](int q) {
        const ent2_t e = sload_entry2(sp + 2 * q);
        return t0 + e[0] < a.in_hi && t0 + e[1] > a.in_lo;
      };
      while (p_lo <= p_hi && !live(p_lo)) ++p_lo;
      while (p_hi > p_lo && !live(p_hi)) --p_hi;
      if (p_lo > 0) {
        toff = (uint32_t)((p_lo * CC + (PF ? 2 : 1)) * WI * 4);
        ea = sbload_t<E>(trs, (uint32_t)(p_lo * CC * WI * 4));
        if (PF) eb = sbload_t<E>(trs, (uint32_t)((p_lo * CC + 1) * WI * 4));
      }
    }
  }
  if (NBUF == 2 && p_lo <= p_hi) {
    __syncthreads();  // a previous tile of this block is done with the LDS rows
    stage_f32_async<NWAVE, ROWCAP>(wave, lds4 + (p_lo & 1) * CC * (ROWCAP / 4), in, a, blk, p_lo * CC,
                                   min(CC, a.rows_in - p_lo * CC), t0);
    if (WEIGHTED) stg_cur = stage_entries<NWAVE, CC>(wave, blk, w_in, a.rows_in, p_lo * CC);
    if (p_lo < p_hi) stg = stage_entries<NWAVE, CC>(wave, blk, w_in, a.rows_in, (p_lo + 1) * CC);
  }
  for (int p = p_lo; p <= p_hi; ++p) {
    const int c0 = p * CC;
    const int ncc = min(CC, a.rows_in - c0);
    const int bufrow = NBUF == 2 ? (p & 1) * CC : 0;
    if (NBUF == 1) {
      __syncthreads();  // the previous pass is done with the LDS rows
      stage_f32<NWAVE, ROWCAP, WEIGHTED>(wave, lds4, in, a, blk, c0, ncc, t0);
      __syncthreads();
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's rows of pass p have landed
      fix_tail_async<NWAVE, ROWCAP>(wave, lds4 + (p & 1) * CC * (ROWCAP / 4), in, a, blk, c0, ncc, t0);
      if (WEIGHTED) scale_rows<NWAVE, ROWCAP>(wave, lds4 + (p & 1) * CC * (ROWCAP / 4), stg_cur, ncc);
      __syncthreads();  // every wave's have; every wave is done with pass p - 1
      if (p + 1 <= p_hi)
        stage_f32_async_pre<NWAVE, ROWCAP>(wave, lds4 + ((p + 1) & 1) * CC * (ROWCAP / 4), in, a, stg, c0 + CC,
                                           min(CC, a.rows_in - c0 - CC), t0);
      if (WEIGHTED) stg_cur = stg;
      if (p + 2 <= p_hi) stg = stage_entries<NWAVE, CC>(wave, blk, w_in, a.rows_in, c0 + 2 * CC);
    }
    // LDS byte address of this lane's window in the pass's first row slot
    uint32_t row = lds_base + (uint32_t)(lane_fresh() * TP * 4) + (uint32_t)(bufrow * ROWCAP * 4);
    if constexpr (RB) {
      // the rows of the pass, block by block; the table marks the last one
      RowPass<TP, DPW, NWIN, ROWCAP>::run(acc, row, ea, trs, toff);
    } else if constexpr (JMP) {
      // the whole pass in one block, each row's DM slots branching into static adds
      if constexpr (PF)
        JmpPrefetchPass<TP, DPW, NWIN, CC, ROWCAP>::run(acc, row, ncc, ea, eb, trs, toff);
      else
        JmpPass<TP, DPW, NWIN, CC, false, JMP == 2, ROWCAP>::run(acc, row, ncc, ea, trs, toff, wa, wrs, woff);
    } else if constexpr (HasWinPass<TP, DPW, NWIN, CC>::value) {
      // the whole pass in one block, index mode on throughout
      WinPass<TP, DPW, NWIN, CC, false, ROWCAP>::run(acc, row, ncc, ea, trs, toff, wa, wrs, woff);
    } else {
      // two rows per iteration with the entry registers swapping roles, so
      // the next row's entry needs no copy
      int cl = 0;
      for (; cl + 1 < ncc; cl += 2) {
        win_step<TP, DPW, NWIN, false>(acc, row + (uint32_t)ea[0] * 4u, ea, eb, trs, toff, wa, wb, wrs, woff);
        row += ROWCAP * 4;
        win_step<TP, DPW, NWIN, false>(acc, row + (uint32_t)eb[0] * 4u, eb, ea, trs, toff, wb, wa, wrs, woff);
        row += ROWCAP * 4;
      }
      if (cl < ncc) {
        win_step<TP, DPW, NWIN, false>(acc, row + (uint32_t)ea[0] * 4u, ea, eb, trs, toff, wa, wb, wrs, woff);
        ea = eb;
        wa = wb;
      }
    }
  }

  if constexpr (DET)
    det_store_f32<TP, DPW, NWAVE>(wave, a, acc, tt, rt, beam, t0);
  else
    win_store<TP, DPW, NWAVE, ADJ>(wave, a, acc, tt, rt, beam);
}

// Waves per SIMD that a jump-form variant's registers allow (its accumulators
// start at JmpAcc0, the window follows them), asked of the compiler so that it
// keeps the rest of the kernel within that budget; 1 (no request) otherwise,
// and for the search epilogue, whose registers would otherwise spill.
template <int TP, int DPW, int NWIN, int CC, int JMP, bool DET = false>
constexpr int win_waves_per_eu() {
  if constexpr (JMP != 0 && !DET) {
    constexpr int regs = (JmpAcc0<TP, DPW, NWIN, CC>::value + TP * DPW + NWIN + 7) / 8 * 8;
    return 512 / regs > 8 ? 8 : 512 / regs;
  } else {
    return 1;
  }
}

template <int TP, int DPW, int NWAVE, int NWIN, int CC, int ROWCAP, int NBUF, bool WEIGHTED, bool ADJ,
          bool DET = false, int JMP = 0>
__global__ __launch_bounds__(64 * NWAVE)
__attribute__((amdgpu_waves_per_eu(win_waves_per_eu<TP, DPW, NWIN, CC, JMP, DET>()))) void win_kernel(TileArgs a) {
  __shared__ float4 lds4[NBUF * CC * ROWCAP / 4];
  const int nblk = a.n_time_tiles * a.n_row_tiles;
  const int W = xcd_remap(blockIdx.x, nblk);
  // Forward: the row tiles of one time tile run on one XCD (they share its
  // input window in that L2).  Adjoint: the time tiles of one row tile do
  // instead, so that the passes skipped near both ends of the output (see
  // win_tile) are spread over every XCD rather than idling the first and last.
  const int tt = ADJ ? W % a.n_time_tiles : W / a.n_row_tiles;
  const int rt = ADJ ? W / a.n_time_tiles : W % a.n_row_tiles;
  win_tile<TP, DPW, NWAVE, NWIN, CC, ROWCAP, NBUF, WEIGHTED, ADJ, DET, JMP>(wave_id(), a, tt, rt, blockIdx.y, lds4);
}

// Persistent form for batches of beams.  The work table is split into one
// queue per XCD (all row tiles of a (beam, time tile) in the same queue, so
// the blocks sharing that input window share that XCD's L2).  Blocks are
// dispatched round-robin over the XCDs, so block i drains queue i % NXCD
// first and then helps the others, in order, until every queue is empty.
// Every beam shares the variant; per-beam pointers and tables come from its
// descriptor.  The counters (one per queue, 128 bytes apart) are cleared by a
// separate kernel before each launch.
template <int TP, int DPW, int NWAVE, int NWIN, int CC, int ROWCAP, int NBUF, bool WEIGHTED, int JMP>
__global__ __launch_bounds__(64 * NWAVE) __attribute__((amdgpu_waves_per_eu(win_waves_per_eu<TP, DPW, NWIN, CC, JMP>())))
void win_persistent(const BeamDesc* __restrict__ beams,
                                                             const int32_t* __restrict__ order,
                                                             const int32_t* __restrict__ qoff, int* counters) {
  __shared__ float4 lds4[NBUF * CC * ROWCAP / 4];
  __shared__ int s_tile;
  const int home = blockIdx.x % kNumXcd;
  const int wave = wave_id();
  for (int qi = 0; qi < kNumXcd; ++qi) {
    const int q = (home + qi) % kNumXcd;
    const int q0 = qoff[q], n = qoff[q + 1] - q0;
    for (;;) {
      __syncthreads();  // everyone is done with s_tile and the LDS rows
      if (wave == 0 && lane_fresh() == 0) s_tile = atomicAdd(counters + q * kCounterStride, 1);
      __syncthreads();
      const int k = __builtin_amdgcn_readfirstlane(s_tile);
      if (k >= n) break;
      const int b = order[2 * (q0 + k)];
      const int local = order[2 * (q0 + k) + 1];
      const TileArgs& a = beams[b].a;
      const int tt = local / a.n_row_tiles, rt = local % a.n_row_tiles;
      win_tile<TP, DPW, NWAVE, NWIN, CC, ROWCAP, NBUF, WEIGHTED, false, false, JMP>(wave, a, tt, rt, 0, lds4);
    }
  }
}

// ---------------------------------------------------------------------------
// Variants.
// ---------------------------------------------------------------------------
// (index, TP samples per lane, DPW rows per wave, NWAVE, NWIN window registers,
//  CC rows per LDS pass, ROWCAP floats per LDS row, NBUF LDS buffers, JMP)
// JMP = 1: each row's DM slots branch into static blocks of adds (JmpPass)
// instead of indexing the window registers; JMP = 2: the same, every row
// reading the whole window (no per-row read-count branches); JMP = 3: one block of
// code per row (RowPass); JMP = 4: as 1 without the next row's window read ahead.
// A lane owns TP consecutive samples; TP/4 odd (12, 20, 28, 36) keeps its
// 16-byte LDS reads free of bank conflicts.
#define F32_VARIANTS(X)                                          \
  X(0, 12, 4, 4, 36, 8, 1024, 1, 0)   /* 16 DMs x 768             */ \
  X(1, 12, 4, 4, 48, 8, 1024, 1, 0)   /* 16 DMs x 768, wide spans */ \
  X(2, 8, 8, 4, 64, 8, 1024, 1, 0)    /* 32 DMs x 512             */ \
  X(3, 16, 8, 4, 72, 8, 2048, 1, 0)   /* 32 DMs x 1024            */ \
  X(4, 8, 4, 4, 48, 16, 1024, 1, 0)   /* 16 DMs x 512             */ \
  X(5, 16, 4, 4, 64, 8, 2048, 1, 0)   /* 16 DMs x 1024            */ \
  X(6, 12, 4, 4, 36, 4, 1024, 2, 0)   /* 16 DMs x 768, async      */ \
  X(7, 12, 8, 4, 56, 4, 1024, 2, 0)   /* 32 DMs x 768, async      */ \
  X(8, 20, 4, 4, 44, 4, 1536, 2, 0)   /* 16 DMs x 1280, async     */ \
  X(9, 12, 4, 8, 36, 4, 1024, 2, 0)   /* 32 DMs x 768, async      */ \
  X(10, 12, 8, 8, 56, 4, 1280, 2, 0)  /* 64 DMs x 768, async      */ \
  X(11, 12, 4, 4, 48, 4, 1024, 2, 0)  /* 16 DMs x 768, async      */ \
  X(12, 8, 8, 4, 64, 4, 1024, 2, 0)   /* 32 DMs x 512, async      */ \
  X(13, 20, 8, 4, 56, 4, 1536, 2, 0)  /* 32 DMs x 1280, async     */ \
  X(14, 28, 4, 4, 48, 4, 2048, 2, 0)  /* 16 DMs x 1792, async     */ \
  X(15, 20, 8, 8, 56, 4, 1792, 2, 0)  /* 64 DMs x 1280, async     */ \
  X(16, 28, 4, 8, 48, 4, 2048, 2, 0)  /* 32 DMs x 1792, async     */ \
  X(17, 20, 8, 8, 56, 8, 1792, 2, 0)  /* 64 DMs x 1280, async     */ \
  X(18, 20, 8, 4, 56, 6, 1536, 2, 0)  /* 32 DMs x 1280, async     */ \
  X(19, 20, 4, 6, 44, 4, 1536, 2, 1)  /* 24 DMs x 1280, jump      */ \
  X(20, 20, 4, 4, 44, 4, 1536, 2, 1)  /* 16 DMs x 1280, jump      */ \
  X(21, 20, 4, 12, 44, 4, 1792, 2, 1) /* 48 DMs x 1280, jump      */ \
  X(22, 20, 8, 4, 56, 6, 1536, 2, 1)  /* 32 DMs x 1280, jump      */ \
  X(23, 20, 8, 8, 56, 4, 1792, 2, 1)  /* 64 DMs x 1280, jump      */ \
  X(24, 28, 4, 4, 48, 4, 2048, 2, 1)  /* 16 DMs x 1792, jump      */ \
  X(25, 28, 4, 8, 48, 4, 2048, 2, 1)  /* 32 DMs x 1792, jump      */ \
  X(26, 12, 4, 8, 36, 4, 1024, 2, 1)  /* 32 DMs x 768, jump       */ \
  X(27, 12, 4, 12, 36, 4, 1024, 2, 1) /* 48 DMs x 768, jump       */ \
  X(28, 20, 8, 4, 56, 6, 1536, 2, 2)  /* 32 DMs x 1280, jump full */ \
  X(29, 20, 4, 12, 44, 4, 1792, 2, 2) /* 48 DMs x 1280, jump full */ \
  X(30, 20, 4, 4, 44, 4, 1536, 2, 2)  /* 16 DMs x 1280, jump full */ \
  X(31, 20, 8, 8, 56, 4, 1792, 2, 2)  /* 64 DMs x 1280, jump full */ \
  X(32, 20, 4, 8, 40, 6, 1536, 2, 3)  /* 32 DMs x 1280, row blocks, 4 waves/SIMD */ \
  X(33, 20, 4, 4, 40, 3, 1536, 2, 3)  /* 16 DMs x 1280, row blocks, 4 waves/SIMD */ \
  X(34, 20, 4, 16, 40, 8, 1792, 2, 3) /* 64 DMs x 1280, row blocks, 4 waves/SIMD */ \
  X(35, 20, 4, 16, 40, 10, 1792, 2, 3) /* 64 DMs x 1280, row blocks, 4 waves/SIMD */ \
  X(36, 20, 4, 16, 40, 8, 1792, 2, 2) /* 64 DMs x 1280, jump full, 4 waves/SIMD */ \
  X(37, 20, 4, 16, 44, 10, 1792, 2, 3) /* 64 DMs x 1280, row blocks, 4 waves/SIMD */ \
  X(38, 20, 4, 16, 44, 8, 1792, 2, 3) /* 64 DMs x 1280, row blocks, 4 waves/SIMD */ \
  X(39, 20, 4, 12, 84, 8, 2304, 2, 1) /* 48 DMs x 1280, jump, wide spans, 3 waves/SIMD */ \
  X(40, 20, 4, 4, 84, 3, 1792, 2, 1)  /* 16 DMs x 1280, jump, wide spans, 3 waves/SIMD */ \
  X(41, 20, 4, 12, 40, 10, 1792, 2, 3) /* 48 DMs x 1280, row blocks */ \
  X(42, 20, 4, 12, 44, 10, 1792, 2, 3) /* 48 DMs x 1280, row blocks */ \
  X(43, 12, 4, 8, 32, 8, 1024, 2, 3) /* 32 DMs x 768, row blocks */ \
  X(49, 20, 4, 16, 40, 10, 1792, 2, 4) /* 64 DMs x 1280, jump: 35 for lists without row patterns */ \
  X(50, 20, 4, 16, 44, 10, 1792, 2, 4) /* 64 DMs x 1280, jump: 37 for lists without row patterns */

}  // namespace dd
