// gfx950 tile kernels of the uint8 path: uint8 rows in, exact int32 sums out
// (or searched in place).  The parallel structure is the one engine.hip
// describes: a block owns a tile of output rows x time samples and stages the
// windows of the input rows it needs in LDS, pass by pass.
#include "detect_dev.h"
#include "device_util.h"
#include "internal.h"

namespace dd {

// ---------------------------------------------------------------------------
// What a uint8 tile does with its sums.  A lane holds Q pieces of four
// consecutive sums of each of the wave's rows: sums(jj, q, s4) gives piece q of
// row jj, place(jj, q) its first sample in the tile (a multiple of 4).
// ---------------------------------------------------------------------------

// Store: non-temporal 16-byte stores, the dominant traffic of the path.
template <int Q, int DPW, int NWAVE, typename SUMS, typename PLACE>
__device__ __forceinline__ void u8_store_tile(const TileArgs& a, int wave, int rt, int beam, int t0, SUMS&& sums,
                                              PLACE&& place) {
  int32_t* out = static_cast<int32_t*>(a.out) + (int64_t)beam * a.out_beam_stride;
#pragma unroll
  for (int jj = 0; jj < DPW; ++jj) {
    const int r = rt * NWAVE * DPW + wave * DPW + jj;
    if (r < a.rows_out) {
      int32_t* orow = out + (int64_t)r * a.out_stride;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        int s4[4];
        sums(jj, q, s4);
        const int t = t0 + place(jj, q);
        if (t + 4 <= a.nout) {
          __builtin_nontemporal_store(s4[0], orow + t + 0);
          __builtin_nontemporal_store(s4[1], orow + t + 1);
          __builtin_nontemporal_store(s4[2], orow + t + 2);
          __builtin_nontemporal_store(s4[3], orow + t + 3);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (t + e < a.nout) orow[t + e] = s4[e];
        }
      }
    }
  }
}

// Single-pulse search in place of the store (see detect_dev.h): each wave
// passes its rows one at a time through its own LDS slot, to give every lane L consecutive samples (the 16-byte chunks are
// XOR-swizzled within groups of eight so that both the writes and the reads
// are free of bank conflicts); the look-ahead comes from the lanes above.
template <int Q, int DPW, int NWAVE, typename SUMS, typename PLACE>
__device__ __forceinline__ void u8_search_tile(const TileArgs& a, uint4* lds, int wave, int lane, int tt, int rt, int beam,
                                               int t0, SUMS&& sums, PLACE&& place) {
  constexpr int ST = 256 * Q;
  constexpr int L = 4 * Q;
  constexpr int IB = Q == 2 ? 3 : Q == 4 ? 4 : 5;
  static_assert((1 << IB) == L, "a lane's run is a power of two");
  __syncthreads();  // every wave is done with the staged rows
  int4* slot = reinterpret_cast<int4*>(lds) + wave * (ST / 4);
  const int nvalid = min(ST, a.det_nsamp - t0);
  const int pos0 = L * lane;
  const bool owned = pos0 < a.tile_step;
  const int lim = nvalid - pos0;
  // While a window's sum (at most 32 samples) leaves room for its start in 31 bits, the records
  // of up to four rows are reduced over the lanes together: 0.57 against 0.62 ms with
  // six maxima and two sums per row one after the other (32 channels, 2048 DM trials, 200,000
  // samples, of which the sums and their way through LDS take 0.38 ms).
  constexpr int G = DPW < 4 ? DPW : 4;
  const int r0 = rt * NWAVE * DPW + wave * DPW;
  const bool together = a.rows_in < (1 << (25 - IB)) / (32 * 255);
  int keys[kDetNW * G];
  double mom[2 * G];
#pragma unroll
  for (int k = 0; k < kDetNW * G; ++k) keys[k] = -1;
#pragma unroll
  for (int k = 0; k < 2 * G; ++k) mom[k] = 0.0;
#pragma unroll
  for (int jj = 0; jj < DPW; ++jj) {
    const int r = r0 + jj;
    DetRec* rec = a.det + ((int64_t)beam * a.rows_out + r) * a.n_time_tiles + tt;
    if (r < a.rows_out) {
      __builtin_amdgcn_sched_barrier(0);  // one row at a time: keeps the search's registers to one row's
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        int s4[4];
        sums(jj, q, s4);
        const int m = place(jj, q) >> 2;  // chunk of samples 4m .. 4m + 3
        slot[m ^ ((m >> 2) & 7)] = make_int4(s4[0], s4[1], s4[2], s4[3]);
      }
      __builtin_amdgcn_wave_barrier();
      int v[L];
#pragma unroll
      for (int c = 0; c < L / 4; ++c) {
        const int m = (L / 4) * lane + c;
        const int4 x = slot[m ^ ((m >> 2) & 7)];
        v[4 * c + 0] = x.x;
        v[4 * c + 1] = x.y;
        v[4 * c + 2] = x.z;
        v[4 * c + 3] = x.w;
      }
      int key[kDetNW];
      double s1, s2;
      if (nvalid < ST)
        det_lane_int<L, IB, true>(v, owned, lim, a.det_s2_u32 != 0, key, s1, s2);
      else
        det_lane_int<L, IB, false>(v, owned, lim, a.det_s2_u32 != 0, key, s1, s2);
      if (together) {
        const int g = jj % G;
#pragma unroll
        for (int k = 0; k < kDetNW; ++k)
          keys[k * G + g] = key[k] < 0 ? -1 : (key[k] >> IB << (IB + 6)) + ((63 - lane) << IB) + (key[k] & (L - 1));
        mom[g] = s1;
        mom[G + g] = s2;
      } else {
        det_commit_int<L, IB>(rec, key, s1, s2, pos0, t0);
      }
      __builtin_amdgcn_wave_barrier();
    }
    // (rows past the end leave the group's values as they were, unwritten)
    const int g = jj % G;
    if (together && g == G - 1 && r - g < a.rows_out)
      det_commit_rows<L, IB, G>(rec - g * a.n_time_tiles, a.n_time_tiles, min(G, a.rows_out - (r - g)), keys, mom, t0);
  }
}

// ---------------------------------------------------------------------------
// uint8 -> int32 tile engine.  Lane l owns 4 consecutive samples in each of
// Q groups spaced 256 samples apart, so its LDS reads of one group are
// consecutive across lanes (no bank conflicts).  Per (input row, output row)
// the lane reads the dword holding its 4 samples and the next one, aligns
// them by the delay's byte offset and adds the 4 bytes into 4 int32
// accumulators.  The output store is the dominant traffic, written with
// non-temporal 16-byte stores.
// ---------------------------------------------------------------------------
template <int NWAVE, int ROWCAP>
__device__ __forceinline__ void stage_u8(uint4* lds, const uint8_t* in, const TileArgs& a, const int32_t* blk, int c0,
                                         int ncc, int t0) {
  const int wave = wave_id(), lane = threadIdx.x & 63;
  for (int cl = wave; cl < ncc; cl += NWAVE) {
    const int sb = blk[2 * (c0 + cl)];
    const int sl = blk[2 * (c0 + cl) + 1];
    const uint8_t* src = in + (int64_t)(c0 + cl) * a.in_stride;
    const int u0 = t0 + sb;
    uint4* dst = lds + cl * (ROWCAP / 16);
    const int nv = sl >> 4;
#pragma unroll 2
    for (int v = lane; v < nv; v += 64) {
      const int u = u0 + 16 * v;
      uint4 x;
      if (u + 16 <= a.in_hi) {
        x = *reinterpret_cast<const uint4*>(src + u);
      } else {
        uint32_t wv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t acc = 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int uu = u + 4 * q + k;
            const uint32_t byte = (uu < a.in_hi) ? (uint32_t)src[uu] : 0u;
            acc |= byte << (8 * k);
          }
          wv[q] = acc;
        }
        x = make_uint4(wv[0], wv[1], wv[2], wv[3]);
      }
      dst[v] = x;
    }
  }
}

// Staging of four byte-shifted copies of each row: copy s holds row[k + s]
// at position k, so a dword holding four consecutive samples starting at any
// byte offset o is the aligned dword (o >> 2) of copy o & 3.  The copies need
// a byte shift, so the data passes through registers: load() fetches a pass's
// bytes into registers, store() writes the shifted copies to LDS.  The kernel calls load() for pass p + 1 before it
// sums pass p, so the global loads are in flight during the adds.
// With fewer rows than waves, the G = NWAVE / CC waves of a row take its
// 16-byte chunks in turn (wave w: row w mod CC, chunks lane + 64 (w / CC +
// G i)), so that every wave stages and each holds fewer chunks.
template <int NWAVE, int CC, int ROWCAP, uint32_t FLIP = 0>
struct ShiftStage {
  static constexpr int G = CC < NWAVE ? NWAVE / CC : 1;  // waves per row
  static_assert(CC >= NWAVE || NWAVE % CC == 0, "rows per pass must divide the waves");
  static constexpr int RPW = (CC + NWAVE - 1) / NWAVE;        // rows staged per wave
  static constexpr int VPL = (ROWCAP / 16 + 64 * G - 1) / (64 * G);  // 16-byte chunks per lane per row
  uint32_t d[RPW][VPL][5];
  int nv[RPW];

  static __device__ __forceinline__ int row_of(int wave, int r) { return G > 1 ? wave % CC : wave + r * NWAVE; }
  static __device__ __forceinline__ int chunk_of(int wave, int lane, int i) {
    return G > 1 ? lane + 64 * (wave / CC + G * i) : lane + 64 * i;
  }

  __device__ __forceinline__ void load(const uint8_t* in, const TileArgs& a, const int32_t* blk, int c0, int ncc,
                                       int t0) {
    const int wave = wave_id(), lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const int cl = row_of(wave, r);
      nv[r] = 0;
      if (cl < ncc) {
        const ent2_t bl = sload_entry2(blk + 2 * (c0 + cl));
        // the row's bytes as a buffer: what lies past its end (rows are a
        // multiple of 16 bytes) reads as zero, without a branch
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(in + (int64_t)(c0 + cl) * a.in_stride), (short)0, a.in_hi, 0x00020000);
        const int u0 = t0 + bl[0];
        nv[r] = bl[1] >> 4;
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
          const int v = chunk_of(wave, lane, i);
          const int u = u0 + 16 * v;
          if (v < nv[r]) {
            const ent4_t x = __builtin_amdgcn_raw_buffer_load_b128(rs, u, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) d[r][i][q] = (uint32_t)x[q];
            d[r][i][4] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, u + 16, 0, 0);
          }
        }
      }
    }
  }

  __device__ __forceinline__ void store(uint4* lds, int ncc) const {
    const int wave = wave_id(), lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const int cl = row_of(wave, r);
#pragma unroll
      for (int i = 0; i < VPL; ++i) {
        const int v = chunk_of(wave, lane, i);
        if (v < nv[r]) {
          uint32_t x[5];
#pragma unroll
          for (int k = 0; k < 5; ++k) x[k] = d[r][i][k] ^ FLIP;
          lds[(0 * CC + cl) * (ROWCAP / 16) + v] = make_uint4(x[0], x[1], x[2], x[3]);
#pragma unroll
          for (int sh = 1; sh < 4; ++sh) {
            lds[(sh * CC + cl) * (ROWCAP / 16) + v] =
                make_uint4(__builtin_amdgcn_alignbyte(x[1], x[0], sh), __builtin_amdgcn_alignbyte(x[2], x[1], sh),
                           __builtin_amdgcn_alignbyte(x[3], x[2], sh), __builtin_amdgcn_alignbyte(x[4], x[3], sh));
          }
        }
      }
    }
    (void)ncc;
  }
};

// Asynchronous staging of one pass: the rows (16-byte buffer loads writing
// LDS directly; positions past the row end read as zero) and this wave's
// table entries for the pass (one 16-byte entry per lane, lanes past the
// pass read zero into the slack of the per-wave table slot).
template <int NWAVE, int ROWCAP>
__device__ __forceinline__ void stage_u8_async(uint4* lds, ent4_t* tabw, const uint8_t* in, const TileArgs& a,
                                               const int32_t* blk, const int32_t* wav, int c0, int ncc, int t0) {
  const int wave = wave_id(), lane = threadIdx.x & 63;
  for (int cl = wave; cl < ncc; cl += NWAVE) {
    const ent2_t bl = sload_entry2(blk + 2 * (c0 + cl));
    const uint8_t* row = in + (int64_t)(c0 + cl) * a.in_stride;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)row, (short)0, a.in_hi, 0x00020000);
    const int u0 = t0 + bl[0];
    const int nv = bl[1] >> 4;
    for (int v0 = 0; v0 < nv; v0 += 64) {
      if (v0 + lane < nv)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LDS_AS void*)(lds + cl * (ROWCAP / 16) + v0), 16,
                                                 u0 + 16 * (v0 + lane), 0, 0, 0);
    }
  }
  const __amdgpu_buffer_rsrc_t rt =
      __builtin_amdgcn_make_buffer_rsrc((void*)(wav + (size_t)c0 * 4), (short)0, ncc * 16, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rt, (LDS_AS void*)tabw, 16, lane * 16, 0, 0, 0);
}

// One block walks `tiles_per_block` consecutive time tiles of one DM tile.
// NBUF = 1: synchronous staging; NBUF = 2: the rows of the next (time tile,
// pass) step are loaded into the second buffer while the current one is
// summed, and the finished tile's stores drain behind the next tile's work.
template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, int NBUF>
__global__ __launch_bounds__(64 * NWAVE) void u8_kernel(TileArgs a) {
  constexpr int ST = 256 * Q;
  constexpr int DT = NWAVE * DPW;
  constexpr int WI = 4;  // packed 16-bit offsets, DPW <= 8
  static_assert(DPW <= 8, "uint8 variants pack at most 8 offsets");
  typedef ent4_t E;
  __shared__ uint4 lds[NBUF * CC * ROWCAP / 16];
  __shared__ E tab[NBUF][NWAVE][NBUF == 2 ? 64 : CC];
  const int tpb = NBUF == 2 ? a.tiles_per_block : 1;
  const int ngroups = (a.n_time_tiles + tpb - 1) / tpb;
  const int nblk = ngroups * a.n_row_tiles;
  const int W = xcd_remap(blockIdx.x, nblk);
  const int grp = W / a.n_row_tiles, rt = W % a.n_row_tiles;
  const int tt0 = grp * tpb;
  const int ntile = min(tpb, a.n_time_tiles - tt0);
  const int beam = blockIdx.y;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int wt = rt * NWAVE + wave;
  const uint8_t* in = static_cast<const uint8_t*>(a.in) + (int64_t)beam * a.in_beam_stride;
  const int32_t* blk = uniform_ptr(a.blk + (size_t)rt * a.rows_in * 2);
  const int32_t* __restrict__ wav = uniform_ptr(a.wav + (size_t)wt * a.rows_in * WI);
  const uint32_t* lds32 = reinterpret_cast<const uint32_t*>(lds);
  int32_t* out = static_cast<int32_t*>(a.out) + (int64_t)beam * a.out_beam_stride;
  const int npass = (a.rows_in + CC - 1) / CC;
  const int nsteps = ntile * npass;

  int acc[DPW][Q][4];
#pragma unroll
  for (int j = 0; j < DPW; ++j)
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[j][q][k] = 0;

  if (NBUF == 2) stage_u8_async<NWAVE, ROWCAP>(lds, tab[0][wave], in, a, blk, wav, 0, min(CC, a.rows_in), tt0 * ST);
  for (int s = 0; s < nsteps; ++s) {
    const int k = s / npass, p = s - k * npass;
    const int t0 = (tt0 + k) * ST;
    const int c0 = p * CC;
    const int ncc = min(CC, a.rows_in - c0);
    const int buf = NBUF == 2 ? (s & 1) : 0;
    if (NBUF == 1) {
      // The wave's offsets for the rows of a pass are copied into LDS with
      // the rows.
      __syncthreads();
      stage_u8<NWAVE, ROWCAP>(lds, in, a, blk, c0, ncc, t0);
      if (lane < ncc) tab[0][wave][lane] = *reinterpret_cast<const E*>(wav + (size_t)(c0 + lane) * WI);
      __syncthreads();
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (s + 1 < nsteps) {
        const int k1 = (s + 1) / npass, p1 = s + 1 - k1 * npass;
        stage_u8_async<NWAVE, ROWCAP>(lds + ((s + 1) & 1) * CC * (ROWCAP / 16), tab[(s + 1) & 1][wave], in, a, blk,
                                      wav, p1 * CC, min(CC, a.rows_in - p1 * CC), (tt0 + k1) * ST);
      }
    }
    const uint32_t* rows = lds32 + buf * CC * (ROWCAP / 4);
    E cur = tab[buf][wave][0];
    for (int cl = 0; cl < ncc; ++cl) {
      // each step reads the next row's entry (a broadcast LDS read) one step
      // ahead of its use
      const E nxt = tab[buf][wave][min(cl + 1, ncc - 1)];
      const uint32_t* row = rows + cl * (ROWCAP / 4);
      uint32_t cw[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) cw[q] = (uint32_t)__builtin_amdgcn_readfirstlane(cur[q]);
#pragma unroll
      for (int jj = 0; jj < DPW; ++jj) {
        const uint32_t o = (cw[jj >> 1] >> (16 * (jj & 1))) & 0xFFFFu;
        const uint32_t sh = o & 3u;
        const uint32_t* pr = row + (o >> 2) + lane;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const uint32_t d0 = pr[64 * q];
          const uint32_t d1 = pr[64 * q + 1];
          const uint32_t v = __builtin_amdgcn_alignbyte(d1, d0, sh);
          acc[jj][q][0] += (int)(v & 0xFFu);
          acc[jj][q][1] += (int)((v >> 8) & 0xFFu);
          acc[jj][q][2] += (int)((v >> 16) & 0xFFu);
          acc[jj][q][3] += (int)(v >> 24);
        }
      }
      cur = nxt;
    }
    if (p == npass - 1) {
#pragma unroll
      for (int jj = 0; jj < DPW; ++jj) {
        const int r = rt * DT + wave * DPW + jj;
        if (r < a.rows_out) {
          int32_t* orow = out + (int64_t)r * a.out_stride;
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int t = t0 + 4 * lane + 256 * q;
            if (t + 4 <= a.nout) {
              __builtin_nontemporal_store(acc[jj][q][0], orow + t + 0);
              __builtin_nontemporal_store(acc[jj][q][1], orow + t + 1);
              __builtin_nontemporal_store(acc[jj][q][2], orow + t + 2);
              __builtin_nontemporal_store(acc[jj][q][3], orow + t + 3);
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (t + e < a.nout) orow[t + e] = acc[jj][q][e];
            }
          }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[jj][q][e] = 0;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// uint8 -> int32 tile engine on byte-shifted rows.  Each input row is staged
// as four copies shifted by 0..3 bytes (ShiftStage), so the four samples
// a lane needs at any delay are one aligned LDS dword: one 4-byte LDS read
// per 4 adds.  The table gives, per (wave tile, input row), each output row's
// dword offset into the staged copies, so a read costs one address add.
// For a dword v = (b0, b1, b2, b3) the lane keeps two sums over rows:
//   E += v & 0x00FF00FF     (16-bit lanes: sum b0, sum b2)
//   U += v >> 8             (sum b1 + 2^8 sum b2 + 2^16 sum b3)
// four two-operand integer operations, which issue at the full rate, per 4
// adds.  Over at most 256 rows neither overflows, and
//   sum b0 = E & 0xFFFF, sum b2 = E >> 16, U - 2^8 sum b2 = sum b1 + 2^16 sum b3.
// WIDE variants move these into int32 sums every 256 input rows; the others
// accept at most 256 input rows.  Sums are exact integers, so the order does
// not matter.
// ---------------------------------------------------------------------------
template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, bool WIDE, bool DET>
__device__ __forceinline__ void u8s_tile(const TileArgs& a) {
  constexpr int ST = 256 * Q;
  constexpr int WI = DPW <= 4 ? 4 : 8;  // ints per table entry
  static_assert(DPW == 2 || DPW == 4 || DPW == 8, "unsupported rows per wave");
  static_assert(256 % CC == 0, "a flush every 256 rows must fall on a pass boundary");
  constexpr int LDS_STAGE = 4 * CC * ROWCAP / 16;
  constexpr int LDS_DET = DET ? NWAVE * ST / 4 : 0;
  __shared__ uint4 lds[LDS_STAGE > LDS_DET ? LDS_STAGE : LDS_DET];
  const int nblk = a.n_time_tiles * a.n_row_tiles;
  const int W = xcd_remap(blockIdx.x, nblk);
  const int tt = W / a.n_row_tiles, rt = W % a.n_row_tiles;
  const int beam = blockIdx.y;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int wt = rt * NWAVE + wave;
  const int t0 = DET ? tt * a.tile_step : tt * ST;
  const uint8_t* in = static_cast<const uint8_t*>(a.in) + (int64_t)beam * a.in_beam_stride;
  const int32_t* blk = uniform_ptr(a.blk + (size_t)rt * a.rows_in * 2);
  const int32_t* __restrict__ wav = uniform_ptr(a.wav + (size_t)wt * a.rows_in * WI);
  const uint32_t* lds32 = reinterpret_cast<const uint32_t*>(lds) + lane;
  const int npass = (a.rows_in + CC - 1) / CC;

  uint32_t ev[DPW][Q], hi[DPW][Q];
  int acc[WIDE ? DPW : 1][WIDE ? Q : 1][4];
#pragma unroll
  for (int j = 0; j < DPW; ++j)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      ev[j][q] = hi[j][q] = 0u;
      if (WIDE)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[WIDE ? j : 0][WIDE ? q : 0][k] = 0;
    }

  // the four sample sums of (output row j, dword q) from the packed sums
  auto unpack = [&](int j, int q, int* s4) {
    const uint32_t s2 = ev[j][q] >> 16;
    const uint32_t u = hi[j][q] - (s2 << 8);
    s4[0] = (int)(ev[j][q] & 0xFFFFu);
    s4[1] = (int)(u & 0xFFFFu);
    s4[2] = (int)s2;
    s4[3] = (int)(u >> 16);
  };

  // this wave's table entries, read with scalar loads (past the last row: zero)
  const __amdgpu_buffer_rsrc_t trs =
      __builtin_amdgcn_make_buffer_rsrc((void*)wav, (short)0, a.rows_in * WI * 4, 0x00020000);
  constexpr int NI = CC * WI;  // ints of one pass's entries
  static_assert(NI == 8 || NI % 16 == 0, "a pass's entries are loaded in 8- or 16-int pieces");
  ShiftStage<NWAVE, CC, ROWCAP> stage;
  stage.load(in, a, blk, 0, min(CC, a.rows_in), t0);
  for (int p = 0; p < npass; ++p) {
    const int c0 = p * CC;
    const int ncc = min(CC, a.rows_in - c0);
    int32_t off[NI];
    if constexpr (NI == 8) {
      const ent8_t x = sbload8(trs, (uint32_t)(c0 * WI * 4));
#pragma unroll
      for (int k = 0; k < 8; ++k) off[k] = x[k];
    } else {
#pragma unroll
      for (int k0 = 0; k0 < NI; k0 += 16) {
        const ent16_t x = sbload16(trs, (uint32_t)((c0 * WI + k0) * 4));
#pragma unroll
        for (int k = 0; k < 16; ++k) off[k0 + k] = x[k];
      }
    }
    __syncthreads();  // every wave is done with pass p - 1's rows
    stage.store(lds, ncc);
    __syncthreads();
    if (p + 1 < npass) stage.load(in, a, blk, c0 + CC, min(CC, a.rows_in - c0 - CC), t0);
#pragma unroll
    for (int cl = 0; cl < CC; ++cl) {
      if (cl >= ncc) break;
#pragma unroll
      for (int jj = 0; jj < DPW; ++jj) {
        const uint32_t* pr = reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(lds32) + off[cl * WI + jj]);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const uint32_t v = pr[64 * q];
          ev[jj][q] += v & 0x00FF00FFu;
          hi[jj][q] += v >> 8;
        }
      }
    }
    if (WIDE && (((p + 1) * CC) % 256 == 0 || p == npass - 1)) {
#pragma unroll
      for (int j = 0; j < DPW; ++j)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          int s4[4];
          unpack(j, q, s4);
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[WIDE ? j : 0][WIDE ? q : 0][k] += s4[k];
          ev[j][q] = hi[j][q] = 0u;
        }
    }
  }

  auto sums = [&](int j, int q, int* s4) {
    if (WIDE) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s4[e] = acc[WIDE ? j : 0][WIDE ? q : 0][e];
    } else {
      unpack(j, q, s4);
    }
  };
  auto place = [&](int, int q) { return 4 * lane + 256 * q; };
  if constexpr (DET)
    u8_search_tile<Q, DPW, NWAVE>(a, lds, wave, lane, tt, rt, beam, t0, sums, place);
  else
    u8_store_tile<Q, DPW, NWAVE>(a, wave, rt, beam, t0, sums, place);
}

// WPE > 0 asks the compiler to fit WPE waves per SIMD (512 / WPE registers),
// so that as many blocks as the LDS allows stay resident on a CU.
template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, bool WIDE, int WPE>
__global__ __launch_bounds__(64 * NWAVE) __attribute__((amdgpu_waves_per_eu(WPE > 0 ? WPE : 1))) void u8s_kernel(
    TileArgs a) {
  u8s_tile<Q, DPW, NWAVE, CC, ROWCAP, WIDE, false>(a);
}

// With the single-pulse search in the epilogue (no occupancy request: the
// search needs its registers).
template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, bool WIDE>
__global__ __launch_bounds__(64 * NWAVE) void u8s_det_kernel(TileArgs a) {
  u8s_tile<Q, DPW, NWAVE, CC, ROWCAP, WIDE, true>(a);
}

// ---------------------------------------------------------------------------
// uint8 -> int32 tile engine on byte-shifted rows with the sums on the matrix
// cores.  Rows are staged as four byte-shifted copies (ShiftStage), so the four
// samples a lane needs at any delay are one aligned LDS dword.  The dwords of
// four input rows (16 bytes per lane) are the B operand of one
// v_mfma_i32_16x16x64_i8: lane 16 h + n holds bytes k = 16 h + 4 d + b (byte b of
// row d's dword) of column n, and with
//   A[m][16 h + 4 d + b] = (m == 4 h + b)
// result row m = 4 h + b is the sum over the four rows d of that byte.  A lane
// gets back rows 4 h .. 4 h + 3 of its column: the four sums of its own dwords.
// One instruction thus does the work of 16 vector operations of the packed sums
// at more than twice their rate, with nothing to unpack or flush: the sums
// are int32 throughout.  The instruction multiplies signed bytes, so the rows
// are staged with their top bits flipped (x - 128) and the sums start at
// 128 * rows_in.
//
// What bounds it: LDS, one byte read per add.  A probe of the inner step alone
// (LDS-resident rows, 16 waves per CU) runs at 101 adds/clk/CU, 106 being what the
// reads alone reach; packed sums reach 71, the identity forms of the 4x4x4 and
// 32x32x32 instructions 79 to 82.  The rows are double-buffered, so a pass has one
// barrier.  Measured on 1024 channels, 2048 DM trials, 20,000 samples: 1.06 ms
// against 1.41 ms for the packed sums flushed to int32 (2.00 ms for the shape that
// used to be the default there); on 32 channels, 2048 DM trials, 200,000 samples
// 0.40 to 0.41 ms, level with the packed sums: the 1.64 GB of output bind there.
// ---------------------------------------------------------------------------
template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, bool DET>
__device__ __forceinline__ void u8m_tile(const TileArgs& a) {
  constexpr int ST = 256 * Q;
  constexpr int WI = DPW <= 4 ? 4 : 8;  // ints per table entry
  constexpr int NI = CC * WI;
  typedef int v4i __attribute__((ext_vector_type(4)));
  constexpr int LDS_BUF = 4 * CC * ROWCAP / 16;
  constexpr int LDS_DET = DET ? NWAVE * ST / 4 : 0;
  __shared__ uint4 lds[2 * LDS_BUF > LDS_DET ? 2 * LDS_BUF : LDS_DET];
  const int nblk = a.n_time_tiles * a.n_row_tiles;
  const int W = xcd_remap(blockIdx.x, nblk);
  const int tt = W / a.n_row_tiles, rt = W % a.n_row_tiles;
  const int beam = blockIdx.y;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int wt = rt * NWAVE + wave;
  const int t0 = DET ? tt * a.tile_step : tt * ST;
  const uint8_t* in = static_cast<const uint8_t*>(a.in) + (int64_t)beam * a.in_beam_stride;
  const int32_t* blk = uniform_ptr(a.blk + (size_t)rt * a.rows_in * 2);
  // the wave's table entries (a multiple of CC rows can be read: the table is padded)
  const int32_t* __restrict__ wav = uniform_ptr(a.wav + (size_t)wt * a.rows_in * WI);
  const int npass = (a.rows_in + CC - 1) / CC;
  // A operand: row lane & 15, bytes k = 16 (lane >> 4) + 4 d + b
  const int ident = ((lane >> 2) & 3) == (lane >> 4) ? 1 << (8 * (lane & 3)) : 0;
  static_assert(CC % 4 == 0, "rows are summed four at a time");

  v4i acc[DPW][Q];
#pragma unroll
  for (int j = 0; j < DPW; ++j)
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[j][q] = (v4i)(128 * a.rows_in);

  ShiftStage<NWAVE, CC, ROWCAP, 0x80808080u> stage;
  stage.load(in, a, blk, 0, min(CC, a.rows_in), t0);
  stage.store(lds, min(CC, a.rows_in));
  if (npass > 1) stage.load(in, a, blk, CC, min(CC, a.rows_in - CC), t0);
  for (int p = 0; p < npass; ++p) {
    const int c0 = p * CC;
    const int ncc = min(CC, a.rows_in - c0);
    int32_t off[NI];
#pragma unroll
    for (int k = 0; k < NI; ++k) off[k] = wav[c0 * WI + k];
    __syncthreads();  // pass p's rows are in LDS, and every wave is done with pass p - 1's
    const char* rows = reinterpret_cast<const char*>(lds + (p & 1) * LDS_BUF) + 4 * lane;
    // step u: two pieces of one output row with four input rows.  A step's
    // reads are issued while the step before is summed; the barriers keep the
    // compiler from hoisting more (and spilling).
    constexpr int SQ = Q / 2, NU = CC / 4 * DPW * SQ;
    int x[2][4][2];
    auto read_step = [&](int u) {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int* pr = reinterpret_cast<const int*>(rows + off[(u / (DPW * SQ) * 4 + d) * WI + u / SQ % DPW]);
        x[u & 1][d][0] = pr[64 * (2 * (u % SQ))];
        x[u & 1][d][1] = pr[64 * (2 * (u % SQ) + 1)];
      }
    };
    read_step(0);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      __builtin_amdgcn_sched_barrier(0);
      if (u + 1 < NU) read_step(u + 1);  // past the last input row: some bytes of the buffer, not summed
      const int left = ncc - u / (DPW * SQ) * 4;  // input rows from this group's first on
      v4i ia;
#pragma unroll
      for (int d = 0; d < 4; ++d) ia[d] = d < left ? ident : 0;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const v4i y = {x[u & 1][0][k], x[u & 1][1][k], x[u & 1][2][k], x[u & 1][3][k]};
        v4i& s = acc[u / SQ % DPW][2 * (u % SQ) + k];
        s = __builtin_amdgcn_mfma_i32_16x16x64_i8(ia, y, s, 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (p + 1 < npass) {
      stage.store(lds + ((p + 1) & 1) * LDS_BUF, min(CC, a.rows_in - c0 - CC));
      if (p + 2 < npass) stage.load(in, a, blk, c0 + 2 * CC, min(CC, a.rows_in - c0 - 2 * CC), t0);
    }
  }
  auto sums = [&](int j, int q, int* s4) {
#pragma unroll
    for (int e = 0; e < 4; ++e) s4[e] = acc[j][q][e];
  };
  auto place = [&](int, int q) { return 4 * lane + 256 * q; };
  if constexpr (DET)
    u8_search_tile<Q, DPW, NWAVE>(a, lds, wave, lane, tt, rt, beam, t0, sums, place);
  else
    u8_store_tile<Q, DPW, NWAVE>(a, wave, rt, beam, t0, sums, place);
}

template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, int WPE>
__global__ __launch_bounds__(64 * NWAVE) __attribute__((amdgpu_waves_per_eu(WPE))) void u8m_kernel(TileArgs a) {
  u8m_tile<Q, DPW, NWAVE, CC, ROWCAP, false>(a);
}

template <int Q, int DPW, int NWAVE, int CC, int ROWCAP, int WPE>
__global__ __launch_bounds__(64 * NWAVE) __attribute__((amdgpu_waves_per_eu(WPE))) void u8m_det_kernel(TileArgs a) {
  u8m_tile<Q, DPW, NWAVE, CC, ROWCAP, true>(a);
}

// ---------------------------------------------------------------------------
// Variant tables and launchers.
// ---------------------------------------------------------------------------
// (index, Q dwords per lane, DPW, NWAVE, CC rows per LDS pass, ROWCAP bytes)
#define U8_VARIANTS(X)                                      \
  X(0, 4, 4, 4, 16, 2048, 1) /* 16 DMs x 1024          */   \
  X(1, 4, 2, 4, 32, 1536, 1) /*  8 DMs x 1024          */   \
  X(2, 2, 4, 4, 16, 1536, 1) /* 16 DMs x 512           */   \
  X(3, 4, 4, 4, 32, 2048, 1) /* 16 DMs x 1024          */   \
  X(4, 2, 2, 4, 32, 1024, 1) /*  8 DMs x 512           */   \
  X(5, 4, 8, 4, 16, 4096, 1) /* 32 DMs x 1024          */   \
  X(6, 4, 4, 8, 16, 4096, 1) /* 32 DMs x 1024          */   \
  X(7, 2, 4, 4, 16, 1152, 2) /* 16 DMs x 512, async    */   \
  X(8, 4, 4, 4, 16, 1664, 2) /* 16 DMs x 1024, async   */   \
  X(9, 4, 4, 8, 8, 2304, 2)  /* 32 DMs x 1024, async   */   \
  X(10, 2, 8, 4, 16, 1792, 2) /* 32 DMs x 512, async   */   \
  X(11, 2, 4, 4, 32, 1152, 2) /* 16 DMs x 512, async   */

// Byte-shifted variants: (index, Q, DPW, NWAVE, CC, ROWCAP bytes per copy,
// WIDE, waves per SIMD asked of the compiler or 0)
#define U8S_VARIANTS(X)                                          \
  X(12, 4, 4, 4, 4, 1792, false, 0) /* 16 DMs x 1024      */    \
  X(13, 2, 4, 8, 4, 1792, false, 0) /* 32 DMs x 512       */    \
  X(14, 4, 4, 8, 8, 2304, false, 0) /* 32 DMs x 1024      */    \
  X(15, 4, 8, 4, 4, 2304, false, 0) /* 32 DMs x 1024      */    \
  X(16, 4, 4, 8, 4, 2304, false, 0) /* 32 DMs x 1024      */    \
  X(17, 4, 4, 4, 2, 1792, false, 0) /* 16 DMs x 1024      */    \
  X(18, 4, 4, 4, 4, 1792, true, 0)  /* 16 DMs x 1024, wide */   \
  X(19, 4, 4, 8, 4, 2304, true, 0)  /* 32 DMs x 1024, wide */   \
  X(20, 8, 4, 8, 4, 3328, false, 0) /* 32 DMs x 2048      */    \
  X(21, 4, 8, 8, 4, 3584, false, 0) /* 64 DMs x 1024      */    \
  X(22, 4, 4, 16, 4, 3584, false, 8) /* 64 DMs x 1024, 2 blocks/CU */

// Matrix-core variants: (index, Q, DPW, NWAVE, CC, ROWCAP bytes per copy, waves per SIMD asked for)
#define U8M_VARIANTS(X)                                     \
  X(23, 4, 4, 8, 4, 2304, 4)  /* 32 DMs x 1024 */        \
  X(24, 4, 4, 16, 4, 3584, 4) /* 64 DMs x 1024 */        \
  X(25, 2, 4, 8, 4, 1792, 6)  /* 32 DMs x 512 */         \
  X(26, 2, 2, 8, 8, 768, 6)   /* 16 DMs x 512, short spans */ \
  X(27, 2, 2, 8, 16, 1152, 4) /* 16 DMs x 512, long spans */

const std::vector<Variant>& variants_u8() {
  static const std::vector<Variant> v = [] {
    std::vector<Variant> r;
#define MAKE_U8(ID, Q, DPW, NW, CC, RC, NB)                                                                 \
  r.push_back(Variant{"u8_q" #Q "_dpw" #DPW "_nw" #NW "_cc" #CC "_buf" #NB, KIND_TILE_U8, Q, DPW, NW, 0, CC, RC, NB, \
                      ID});
    U8_VARIANTS(MAKE_U8)
#undef MAKE_U8
#define MAKE_U8S(ID, Q, DPW, NW, CC, RC, WIDE, WPE)                                                          \
  r.push_back(Variant{WIDE        ? "u8s_q" #Q "_dpw" #DPW "_nw" #NW "_cc" #CC "_wide"                          \
                      : WPE > 0   ? "u8s_q" #Q "_dpw" #DPW "_nw" #NW "_cc" #CC "_o" #WPE                        \
                                  : "u8s_q" #Q "_dpw" #DPW "_nw" #NW "_cc" #CC,                                 \
                      KIND_TILE_U8, Q, DPW, NW, 0, CC, RC, 1, ID, WIDE ? 2 : 1});
    U8S_VARIANTS(MAKE_U8S)
#undef MAKE_U8S
#define MAKE_U8M(ID, Q, DPW, NW, CC, RC, WPE)                                                                \
  r.push_back(Variant{"u8m_q" #Q "_dpw" #DPW "_nw" #NW "_cc" #CC "_row" #RC "_buf2", KIND_TILE_U8, Q, DPW, NW, 0, CC, RC, \
                      1, ID, 3});
    U8M_VARIANTS(MAKE_U8M)
#undef MAKE_U8M
    return r;
  }();
  return v;
}

hipError_t launch_tiled_u8(const Variant& v, const TileArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(64 * v.nwave);
#define LAUNCH_U8(ID, Q, DPW, NW, CC, RC, NB)                                          \
  if (v.id == ID) {                                                                    \
    hipLaunchKernelGGL((u8_kernel<Q, DPW, NW, CC, RC, NB>), grid, block, 0, s, a);     \
    return hipGetLastError();                                                          \
  }
  U8_VARIANTS(LAUNCH_U8)
#undef LAUNCH_U8
#define LAUNCH_U8S(ID, Q, DPW, NW, CC, RC, WIDE, WPE)                                       \
  if (v.id == ID) {                                                                         \
    hipLaunchKernelGGL((u8s_kernel<Q, DPW, NW, CC, RC, WIDE, WPE>), grid, block, 0, s, a);  \
    return hipGetLastError();                                                               \
  }
  U8S_VARIANTS(LAUNCH_U8S)
#undef LAUNCH_U8S
#define LAUNCH_U8M(ID, Q, DPW, NW, CC, RC, WPE)                                             \
  if (v.id == ID) {                                                                         \
    hipLaunchKernelGGL((u8m_kernel<Q, DPW, NW, CC, RC, WPE>), grid, block, 0, s, a);        \
    return hipGetLastError();                                                               \
  }
  U8M_VARIANTS(LAUNCH_U8M)
#undef LAUNCH_U8M
  return hipErrorInvalidDeviceFunction;
}

hipError_t launch_detect_u8(const Variant& v, const TileArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(64 * v.nwave);
#define LAUNCH_DU8(ID, Q, DPW, NW, CC, RC, WIDE, WPE)                                     \
  if (v.id == ID) {                                                                       \
    hipLaunchKernelGGL((u8s_det_kernel<Q, DPW, NW, CC, RC, WIDE>), grid, block, 0, s, a); \
    return hipGetLastError();                                                             \
  }
  U8S_VARIANTS(LAUNCH_DU8)
#undef LAUNCH_DU8
#define LAUNCH_DU8M(ID, Q, DPW, NW, CC, RC, WPE)                                              \
  if (v.id == ID) {                                                                           \
    hipLaunchKernelGGL((u8m_det_kernel<Q, DPW, NW, CC, RC, WPE>), grid, block, 0, s, a);      \
    return hipGetLastError();                                                                 \
  }
  U8M_VARIANTS(LAUNCH_DU8M)
#undef LAUNCH_DU8M
  return hipErrorInvalidDeviceFunction;
}

}  // namespace dd
