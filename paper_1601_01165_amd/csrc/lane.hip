// gfx950 FP32 tile kernels for work that leaves the chip short of waves: few
// output rows, short series, or delay spans too wide for the register window.
//
// The register-window kernels (engine.hip) give a wave 80 sums per lane, so a
// call of a few hundred output rows and a few thousand samples has fewer waves
// than the chip has SIMDs, and each wave's chain of input rows runs at the
// latency of its window reads and jumps.  Here a lane holds only 4 Q sums of each
// of DPW output rows and reads every term from LDS (4-byte reads of samples 64
// apart), wherever its row starts.  Rows are staged by 16-byte buffer loads that
// write LDS directly into a ring of NBUF buffers of CC rows; a pass's rows are
// asked for NBUF - 1 passes before they are summed, so the memory latency hides
// behind several short passes, with one barrier per pass.  Nothing depends on how
// the delays of neighbouring output rows relate.  Sums take one term per input
// row in ascending order with one rounding each (a weighted term is the rounded
// product), as everywhere.
//
// What bounds it: with the chip full, the LDS reads, one 4-byte read per add (26
// adds/clk/CU, 2.46 ms on 1024 channels, 2048 DM trials, 20,000 samples, where the
// register-window kernels take 1.04 ms); with about a block per CU, a pass's
// barrier and latency (0.8 us per 8 rows).  301 DM trials x 2003 samples of 1024
// channels: 473 us in 64 x 1280 tiles, 103 us in 8 x 256 ones.  Four copies of each
// row shifted by 0..3 samples, read 16 bytes at a time, were slower everywhere
// (4.54 against 2.46 ms, 201 against 103 us): staging four times the bytes costs
// more than the wider reads save.
#include "device_util.h"
#include "internal.h"

namespace dd {

template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, int NBUF, bool WEIGHTED, bool ADJ>
struct LaneTile {
  static constexpr int ST = 256 * Q;
  static constexpr int DT = NWAVE * DPW;
  static constexpr int RPW = CC / NWAVE;            // rows staged by one wave per pass
  static_assert(CC % NWAVE == 0, "every wave stages the same number of rows");
  static constexpr int NCH = (ROWCAP + 255) / 256;  // loads per row
  static constexpr int PER_PASS = RPW * NCH;        // loads of a wave per pass
  static constexpr int BUF = CC * ROWCAP * 4;       // bytes of one buffer
  static_assert(ROWCAP % 4 == 0 && NBUF >= 2, "rows are staged in 16-byte pieces");

  // Ask for the rows of pass p (rows past the last one are the last row again,
  // so every pass issues PER_PASS loads and the wait below can count them).
  // sb[k]: stage base of the wave's k-th row.
  static __device__ __forceinline__ void stage(int wave, uint32_t lds_base, const float* in, const TileArgs& a,
                                               const int* sb, int p, int t0) {
    const int lane = lane_fresh();
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const int cl = wave * RPW + k;
      const int c = min(p * CC + cl, a.rows_in - 1);
      const float* base = in + (int64_t)c * a.in_stride + a.in_lo + a.in_shift;
      // positions outside [in_lo, in_hi) read as zero, also in a 16-byte piece
      // that straddles in_hi (the range is checked per 4 bytes; tested with NaN in the
      // rows' padding); none straddles in_lo: both it and the pieces are multiples of
      // 16 bytes
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (a.in_hi - a.in_lo) * 4, 0x00020000);
      const int u0 = t0 + sb[k] - a.in_lo;
      const uint32_t dst = lds_base + (uint32_t)((p % NBUF) * BUF + cl * ROWCAP * 4);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const int v = 64 * ch + lane;
        const uint32_t off = (uint32_t)(u0 + 4 * v) * 4u;
        uint32_t m0s;
        // the compiler does not see that this load writes LDS, so it adds no
        // wait of its own before the reads of other buffers
        if (ROWCAP - 256 * ch >= 256 || 4 * v < ROWCAP)
          asm volatile(
              "s_mov_b32 %[m0s], m0\n\t"
              "s_mov_b32 m0, %[dst]\n\t"
              "s_nop 0\n\t"
              "buffer_load_dwordx4 %[off], %[rs], 0 offen lds\n\t"
              "s_mov_b32 m0, %[m0s]"
              : [m0s] "=&s"(m0s)
              : [dst] "s"(dst + 1024 * ch), [off] "v"(off), [rs] "s"(rs)
              : "memory");
      }
    }
  }

  static __device__ __forceinline__ void run(int wave, const TileArgs& a, int tt, int rt, int beam, float4* lds4) {
    tt = __builtin_amdgcn_readfirstlane(tt);
    rt = __builtin_amdgcn_readfirstlane(rt);
    const int t0 = tt * ST;
    const int lane = threadIdx.x & 63;
    const float* in = static_cast<const float*>(a.in) + (int64_t)beam * a.in_beam_stride;
    const const_table<int32_t> blk = uniform_table(a.blk + (size_t)rt * a.rows_in * 2);
    // (a whole pass's entries can be read: the table is padded)
    const const_table<int32_t> wav = uniform_table(a.wav + (size_t)(rt * NWAVE + wave) * a.rows_in * DPW);
    const const_table<float> w_in = uniform_table(a.w_in);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(LDS_AS float4*)(lds4);
    const char* const ldsb = reinterpret_cast<const char*>(lds4);
    const int npass = (a.rows_in + CC - 1) / CC;

    float acc[DPW][4 * Q];
#pragma unroll
    for (int j = 0; j < DPW; ++j)
#pragma unroll
      for (int i = 0; i < 4 * Q; ++i) acc[j][i] = 0.f;

    // the passes that meet the valid samples at all (adjoint)
    int p_lo = 0, p_hi = npass - 1;
    if constexpr (ADJ) {
      if (a.span) {
        const const_table<int32_t> sp = uniform_table(a.span + (size_t)rt * npass * 2);
        auto live = [&](int q) { return t0 + sp[2 * q] < a.in_hi && t0 + sp[2 * q + 1] > a.in_lo; };
        while (p_lo <= p_hi && !live(p_lo)) ++p_lo;
        while (p_hi > p_lo && !live(p_hi)) --p_hi;
      }
    }

    auto bases = [&](int p, int* sb) {
#pragma unroll
      for (int k = 0; k < RPW; ++k) sb[k] = blk[2 * min(p * CC + wave * RPW + k, a.rows_in - 1)];
    };
    // table entries and weights of a pass, loaded (scalar) while the pass before is summed
    int32_t off[CC * DPW], off_n[CC * DPW];
    float wt[CC], wt_n[CC];
    auto entries = [&](int p) {
      const int c0 = min(p * CC, a.rows_in - 1);
#pragma unroll
      for (int k = 0; k < CC * DPW; ++k) off_n[k] = wav[c0 * DPW + k];
      if (WEIGHTED) {
#pragma unroll
        for (int cl = 0; cl < CC; ++cl) wt_n[cl] = w_in[min(c0 + cl, a.rows_in - 1)];
      }
    };
    __syncthreads();  // a previous tile of this block is done with the buffers
    int sb[RPW];
    if (p_lo <= p_hi) {
      for (int p = p_lo; p < p_lo + NBUF - 1; ++p) {
        bases(p, sb);
        stage(wave, lds_base, in, a, sb, p, t0);
      }
      bases(p_lo + NBUF - 1, sb);
      entries(p_lo);
    }
    for (int p = p_lo; p <= p_hi; ++p) {
      const int c0 = p * CC;
      const int ncc = min(CC, a.rows_in - c0);
#pragma unroll
      for (int k = 0; k < CC * DPW; ++k) off[k] = off_n[k];
      if (WEIGHTED) {
#pragma unroll
        for (int cl = 0; cl < CC; ++cl) wt[cl] = wt_n[cl];
      }
      // this wave's rows of pass p have landed (the loads of the NBUF - 2
      // passes after it may still be under way); after the barrier every
      // wave's have, and every wave is done with pass p - 1's buffer
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NBUF - 2) * PER_PASS) : "memory");
      stage(wave, lds_base, in, a, sb, p + NBUF - 1, t0);
      bases(p + NBUF, sb);
      entries(p + 1);
      const char* rows = ldsb + (p % NBUF) * BUF + 4 * lane;
      auto add_row = [&](int cl) {
#pragma unroll
        for (int jj = 0; jj < DPW; ++jj) {
          const char* pr = rows + off[cl * DPW + jj];
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            float x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = reinterpret_cast<const float*>(pr)[256 * q + 64 * i];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float term = WEIGHTED ? wt[cl] * x[i] : x[i];
              acc[jj][4 * q + i] = acc[jj][4 * q + i] + term;
            }
          }
        }
      };
      if (ncc == CC) {
#pragma unroll
        for (int cl = 0; cl < CC; ++cl) add_row(cl);
      } else {
#pragma unroll
        for (int cl = 0; cl < CC - 1; ++cl)
          if (cl < ncc) add_row(cl);
      }
    }
    // the loads asked for past the last pass must land before the buffers are
    // used again or given back
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    float* out = static_cast<float*>(a.out);
#pragma unroll
    for (int jj = 0; jj < DPW; ++jj) {
      const int r = rt * DT + wave * DPW + jj;
      if (r >= a.rows_out) break;
      const float scale = (ADJ && a.w_out) ? a.w_out[r] : 1.f;
      float* orow = out ? out + (int64_t)beam * a.out_beam_stride + (int64_t)r * a.out_stride : nullptr;
      const float* xrow =
          ADJ && a.partial ? a.x + (int64_t)beam * a.x_beam_stride + (int64_t)r * a.x_stride : nullptr;
      double gw = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = t0 + 256 * q + 64 * i + lane;
          if (t < a.nout) {
            if (ADJ && xrow) gw += (double)xrow[t] * (double)acc[jj][4 * q + i];
            if (orow) orow[t] = ADJ ? scale * acc[jj][4 * q + i] : acc[jj][4 * q + i];
          }
        }
      }
      if (ADJ && xrow) {
        // fixed-order reduction over the wave
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) gw += __shfl_xor(gw, m, 64);
        if (lane == 0) a.partial[((size_t)beam * a.n_time_tiles + tt) * a.rows_out + r] = gw;
      }
    }
  }
};

template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, int NBUF, bool WEIGHTED, bool ADJ>
__global__ __launch_bounds__(64 * NWAVE) void lane_kernel(TileArgs a) {
  __shared__ float4 lds4[NBUF * CC * ROWCAP / 4];
  const int W = xcd_remap(blockIdx.x, a.n_time_tiles * a.n_row_tiles);
  const int tt = W / a.n_row_tiles, rt = W % a.n_row_tiles;
  LaneTile<Q, DPW, NWAVE, CC, ROWCAP, NBUF, WEIGHTED, ADJ>::run(wave_id(), a, tt, rt, blockIdx.y, lds4);
}

// (index, Q, DPW, NWAVE, CC rows per pass, ROWCAP floats per row, NBUF)
#define LANE_VARIANTS(X)                                    \
  X(44, 1, 1, 8, 8, 384, 4)  /* 8 DMs x 256 */              \
  X(45, 1, 2, 8, 8, 384, 4)  /* 16 DMs x 256 */             \
  X(46, 2, 2, 8, 8, 768, 3)  /* 16 DMs x 512 */             \
  X(47, 2, 1, 8, 8, 640, 4)  /* 8 DMs x 512 */              \
  X(48, 1, 2, 8, 8, 1024, 3) /* 16 DMs x 256, wide spans */

void lane_variants(std::vector<Variant>& r) {
#define MAKE_LANE(ID, Q, DPW, NW, CC, RC, NB)                                                                   \
  r.push_back(Variant{"lane_q" #Q "_dpw" #DPW "_nw" #NW "_cc" #CC "_row" #RC "_ring" #NB, KIND_LANE_F32, 4 * Q, \
                      DPW, NW, 0, CC, RC, NB, ID});
  LANE_VARIANTS(MAKE_LANE)
#undef MAKE_LANE
}

hipError_t launch_lane(const Variant& v, const TileArgs& a, dim3 grid, bool adjoint, hipStream_t s) {
  const dim3 block(64 * v.nwave);
#define LAUNCH_LANE(ID, Q, DPW, NW, CC, RC, NB)                                                             \
  if (v.id == ID) {                                                                                             \
    if (adjoint) {                                                                                              \
      hipLaunchKernelGGL((lane_kernel<Q, DPW, NW, CC, RC, NB, false, true>), grid, block, 0, s, a);       \
    } else if (a.w_in)                                                                                          \
      hipLaunchKernelGGL((lane_kernel<Q, DPW, NW, CC, RC, NB, true, false>), grid, block, 0, s, a);         \
    else                                                                                                        \
      hipLaunchKernelGGL((lane_kernel<Q, DPW, NW, CC, RC, NB, false, false>), grid, block, 0, s, a);        \
    return hipGetLastError();                                                                                   \
  }
  LANE_VARIANTS(LAUNCH_LANE)
#undef LAUNCH_LANE
  return hipErrorInvalidDeviceFunction;
}

}  // namespace dd
