// Convolution with the input rows cached in LDS as they lie: for filters of any size over any number of channels
// (operator table, Conv2d row: large filters, image inputs of three channels), at any alignment.
//
// GEMM view: m = filter, n = (image, out row, out col), k = (channel, filter row, filter column), the filter columns
// padded to whole 16-byte chunks (8 elements, 4 for fp32).  One chunk of k is then one run of consecutive input
// elements, I[img][c][p * stride - pad + r][q * stride - pad + 0..7], so with the input rows in LDS a lane's B fragment
// is five consecutive dwords shifted by the parity of its first element; no im2col buffer, no transpose and no index
// arithmetic per element.  The columns beyond the filter are cleared in both operands (an infinity in the input next to
// the window must not meet a zero weight).
//
// One LDS stage holds cStageCh channels: the filters [BM][channel, row, chunk] (row pitch an odd number of 16-byte
// chunks: 16 consecutive rows fall into different banks) and, per channel, the stacked rows of the zero-padded images
// that the workgroup's pixels touch.  Rows and columns outside an image are never written and stay zero.
//
// What bounds it: for few channels the output, 16 x 64 x 56 x 56 fp32 from three channels and 7 x 7 filters, 12.8 of
// 14.1 MB, and the latency of one chain of load, LDS, MFMA and store; the element gather that served these layers
// before computed every operand's index: 32.9 -> 9.3 us.  Padding wastes MFMA work (7 of 8 columns are
// used, 5 of 8, 3 of 8), which is why 3 x 3 filters over many channels stay with the channel-last patch.
#pragma once
#include "gemm_kernel.hpp"

namespace gensor {

template <typename T_, typename OutT_, int BM_, int BN_, int WM_, int WN_>
struct ConvRowsCfg {
  typedef T_ T;
  typedef OutT_ OutT;
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, MB = 32;
  static constexpr int ES = ElemSize<T>::value, EPC = 16 / ES;
  static constexpr int WAVES_N = BN / WN, WAVES = BM / WM * WAVES_N, THREADS = WAVES * 64;
  static constexpr int MBLK = WM / MB, NBLK = WN / MB;
  // 16-byte units a thread has in flight: filters, input rows.  Two input rows where a wave has two blocks of 16-bit operands:
  // four spilled 13-15 of the 128 registers that two workgroups of eight such waves per CU leave (16 x 16 x 112 x 112, 64 filters
  // 5x5: 55 -> 49 us; 8 x 40 x 28 x 28: 32 -> 28; five and three, without spills, too: 49, 29.6).
  static constexpr int A_BATCH = 6, P_BATCH = ES == 2 && MBLK * NBLK == 2 ? 2 : 4;
  static_assert(BM % WM == 0 && BN % WN == 0 && WM % MB == 0 && WN % MB == 0, "tiles");
};

// Byte offset of an output pixel's window in the staged rows: first row counted from the stage's first, first column
// counted from the first one in LDS.
__host__ __device__ inline uint32_t rows_window(int row, int col, int row_pitch, int es) { return (uint32_t)(row * row_pitch + col * es); }

// The chunks of a stage relative to a window, in the order channel, filter row, chunk of the row.  An odd number of chunks has one
// more behind the last (the MFMA takes two): it has no rows of its own and is read from the last chunk's, for its value is cleared.
// ONE_CHUNK: a filter row is one chunk.
template <bool ONE_CHUNK>
struct RowsWalk {
  int sc = 0, r = 0;
  uint32_t off = 0;
  __host__ __device__ void advance(int R, int SC, int row_pitch, int chan_pitch) {
    if constexpr (ONE_CHUNK) {
      off += (uint32_t)row_pitch;
    } else {
      off += 16;
      if (++sc < SC) return;
      sc = 0;
      off += (uint32_t)(row_pitch - 16 * SC);
    }
    if (++r == R) { r = 0; off += (uint32_t)(chan_pitch - R * row_pitch); }
  }
  static __host__ __device__ uint32_t last(int channels, int R, int SC, int row_pitch, int chan_pitch) {
    return (uint32_t)((channels - 1) * chan_pitch + (R - 1) * row_pitch + 16 * (SC - 1));
  }
  __host__ __device__ uint32_t at(uint32_t last_off) const { return off < last_off ? off : last_off; }
};

// ONE_CHUNK: a filter row is one chunk (at most 8 columns, 4 for fp32), whose mask is the same throughout.
template <typename C, bool ONE_CHUNK>
__global__ __launch_bounds__(C::THREADS, C::MBLK * C::NBLK > 2 ? 2 : 4) void conv_rows_kernel(const KernelArgs args) {
  typedef typename C::T T;
  typedef Mfma<T, C::MB> MF;
  typedef typename MF::Acc Acc;
  constexpr int ES = C::ES, EPC = C::EPC, BM = C::BM, MB = C::MB, THREADS = C::THREADS;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  GENSOR_LDS char* lds = (GENSOR_LDS char*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave / C::WAVES_N, wave_n = wave % C::WAVES_N;

  const int total = args.tiles_m * args.tiles_n;
  int wg = blockIdx.x;
  // a contiguous range of tiles per XCD; other counts keep the hardware's order (16 x 3 x 112 x 112, 7x7, stride 2: 196 tiles, 9.7 us
  // against 10.2; 2 x 16 x 63 x 30, 5x5: 8.8 against 9.25; nothing gained)
  if ((total & 7) == 0) wg = xcd_contiguous(wg, total);
  int tile_m, tile_n;
  tile_of(args, wg, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * args.cTilePx;
  const int n_end = min(args.N, n0 + args.cTilePx);

  // geometry
  const int Cc = args.cC, H = args.cH, W = args.cW, R = args.cR, S = args.cS, P = args.cP, Q = args.cQ;
  const int stride = args.cStride, pad = args.cPad;
  const int Hp = H + 2 * pad, PQ = P * Q;
  const int SC = (S + EPC - 1) / EPC;                    // chunks per filter row
  const int XO = (pad + EPC - 1) / EPC * EPC;            // LDS column of input column 0: input rows are written as whole chunks
  const int a_pitch = args.cApitch, rows = args.cPatchRows, row_pitch = args.cRowPitch, stage_ch = args.cStageCh;
  const int chan_pitch = rows * row_pitch;
  GENSOR_LDS char* abase = lds;
  GENSOR_LDS char* pbase = lds + BM * a_pitch;
  const int g_first = n0 / Q;
  const int R0 = (g_first / P) * Hp + (g_first % P) * stride;       // first stacked padded input row

  // Operands at any alignment, fetched as the five aligned dwords around a chunk: the descriptor starts on the 16-byte
  // granule of the first element and ends on a dword boundary (see fetch_loose of the contraction kernel).
  constexpr uint32_t RSRC_FLAGS = 0x00020000u, OOB = 0x80000000u;
  auto loose_rsrc = [&](const void* p, int64_t bytes, uint32_t& skew) {
    skew = (uint32_t)((uintptr_t)p & 15u);
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p - skew), 0, (uint32_t)((bytes + skew + 3) & ~3ll), RSRC_FLAGS);
  };
  uint32_t skew_in, skew_w;
  const __amdgpu_buffer_rsrc_t rs_in = loose_rsrc(args.B, args.cInBytes, skew_in);
  const __amdgpu_buffer_rsrc_t rs_w = loose_rsrc(args.A, args.cWBytes, skew_w);
  struct Unit { u32x4 v; uint32_t w; };
  auto load_unit = [&](const __amdgpu_buffer_rsrc_t& r, uint32_t off, Unit& u) {
    u.v = __builtin_amdgcn_raw_buffer_load_b128(r, off & ~3u, 0, 0);
    if constexpr (ES == 2) u.w = __builtin_amdgcn_raw_buffer_load_b32(r, (off & ~3u) + 16u, 0, 0);
  };
  // mask of dword d of a chunk that has `n` valid elements from its start
  auto dword_mask = [](int n, int d) -> uint32_t {
    if constexpr (ES == 4) return n > d ? 0xffffffffu : 0u;
    else return n > 2 * d + 1 ? 0xffffffffu : (n > 2 * d ? 0xffffu : 0u);
  };
  auto unit_value = [&](const Unit& u, uint32_t off, int valid) -> u32x4 {
    u32x4 o;
    const uint32_t d[5] = {u.v[0], u.v[1], u.v[2], u.v[3], u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (ES == 4) o[e] = d[e];
      else o[e] = __builtin_amdgcn_alignbyte(d[e + 1], d[e], off & 2u);
      o[e] &= dword_mask(valid, e);
    }
    return o;
  };

  // u / d by the reciprocal ceil(2^32 / d) the host passed (0 for d = 1): exact while u * d stays below 2^32
  auto divide = [](int u, uint32_t rec) -> int { return rec ? (int)__umulhi((uint32_t)u, rec) : u; };

  // ---- staging.  Filter unit: chunk h of filter m; h counts (channel, filter row, chunk) of a full stage, and one more,
  // all zero, where that count is odd (MFMA takes two chunks at a time).  Input unit: 16 bytes of one stacked row of
  // one channel.  Where a unit comes from and goes to depends on its number alone, so it is worked out once for the
  // first batch of units, which is all of them on most layers, and kept.
  const int segs = (W + EPC - 1) / EPC;
  const int wrow = Cc * R * S;                           // elements of one filter
  const int nch_full = stage_ch * R * SC, nche = (nch_full + 1) & ~1;
  const int a_units = BM * nche, p_units = stage_ch * rows * segs;
  // source: byte offset, or OOB; place: LDS byte offset, with the unit's chunk in its row (filters) in the low bits
  auto filter_unit = [&](int u, int c0, uint32_t& src, int& place) {
    const int m = divide(u, args.cRec[0]), h = u - m * nche;
    const int rho = divide(h, args.cRec[1]), sc = h - rho * SC;
    const bool ok = u < a_units && m0 + m < args.M && h < nch_full && c0 * R + rho < Cc * R;
    src = ok ? skew_w + (uint32_t)(((m0 + m) * wrow + (c0 * R + rho) * S + sc * EPC) * ES) : OOB;
    place = u < a_units ? (m * a_pitch + h * 16) | sc : -1;
  };
  auto input_unit = [&](int u, int c0, uint32_t& src, int& place, int& x) {
    const int t = divide(u, args.cRec[2]), seg = u - t * segs;
    const int c = divide(t, args.cRec[3]);
    const int srow = R0 + t - c * rows;
    const int img = divide(srow, args.cRec[4]), y = srow - img * Hp - pad;
    const bool ok = u < p_units && c0 + c < Cc && img < args.cN && y >= 0 && y < H;
    x = seg * EPC;
    src = ok ? skew_in + (uint32_t)((((img * Cc + c0 + c) * H + y) * W + x) * ES) : OOB;
    place = t * row_pitch + (XO + x) * ES;
  };
  // One batch: all of a thread's loads go out before the first LDS write.  Nothing of it is kept over the products, which
  // leaves registers for two or three waves per SIMD: the other workgroups of the CU cover this one's loads.  (Kept
  // unit positions and the next stage's loads in flight under the products spilled at two waves per SIMD and were slower at one.)
  auto stage = [&](int c0, int batch) {
    uint32_t a_src[C::A_BATCH], p_src[C::P_BATCH];
    int a_place[C::A_BATCH], p_place[C::P_BATCH], p_x[C::P_BATCH];
    Unit ua[C::A_BATCH], up[C::P_BATCH];
    const int a_first = batch * C::A_BATCH * THREADS, p_first = batch * C::P_BATCH * THREADS;
#pragma unroll
    for (int i = 0; i < C::A_BATCH; ++i)
      if (a_first + i * THREADS + wave * 64 < a_units) {
        filter_unit(a_first + i * THREADS + tid, c0, a_src[i], a_place[i]);
        load_unit(rs_w, a_src[i], ua[i]);
      }
#pragma unroll
    for (int i = 0; i < C::P_BATCH; ++i)
      if (p_first + i * THREADS + wave * 64 < p_units) {
        input_unit(p_first + i * THREADS + tid, c0, p_src[i], p_place[i], p_x[i]);
        load_unit(rs_in, p_src[i], up[i]);
      }
#pragma unroll
    for (int i = 0; i < C::A_BATCH; ++i)
      if (a_first + i * THREADS + wave * 64 < a_units && a_place[i] >= 0) {
        const int sc = a_place[i] & 15;
        *(GENSOR_LDS u32x4*)(abase + (a_place[i] - sc)) = unit_value(ua[i], a_src[i], a_src[i] < OOB ? S - sc * EPC : 0);
      }
#pragma unroll
    for (int i = 0; i < C::P_BATCH; ++i)
      // (rows outside the images were out of range and are not written: they stay zero)
      if (p_first + i * THREADS + wave * 64 < p_units && p_src[i] < OOB)
        *(GENSOR_LDS u32x4*)(pbase + p_place[i]) = unit_value(up[i], p_src[i], W - p_x[i]);
  };
  const int batches = max((a_units + C::A_BATCH * THREADS - 1) / (C::A_BATCH * THREADS), (p_units + C::P_BATCH * THREADS - 1) / (C::P_BATCH * THREADS));

  // zero the patch once: what no unit writes stays zero
  for (int o = tid * 16; o < args.cStageBytes - BM * a_pitch; o += THREADS * 16) *(GENSOR_LDS u32x4*)(pbase + o) = u32x4{0u, 0u, 0u, 0u};

  Acc acc[C::MBLK][C::NBLK];
#pragma unroll
  for (int i = 0; i < C::MBLK; ++i)
#pragma unroll
    for (int j = 0; j < C::NBLK; ++j)
#pragma unroll
      for (int v = 0; v < MF::NACC; ++v) acc[i][j][v] = 0.f;

  const int frow = lane % MB, fgrp = lane / MB;
  const bool idle = n0 + wave_n * C::WN >= n_end;        // a wave whose columns all lie beyond the tile's pixels
  uint32_t b_at[C::NBLK], b_odd[C::NBLK];                // the lane's window: byte offset of its first dword, parity
  uint32_t o_at[C::NBLK];                                // its output pixel: element offset at filter 0
#pragma unroll
  for (int bj = 0; bj < C::NBLK; ++bj) {
    const int d = min(wave_n * C::WN + bj * MB + frow, n_end - 1 - n0);
    const int dq = n0 - g_first * Q + d;                 // counted from the first pixel of the tile's first output row
    const int dg = divide(dq, args.cRec[5]), q = dq - dg * Q;
    const int dp = g_first % P + dg;                     // ... and from the first row of its first image
    const int di = divide(dp, args.cRec[6]), p = dp - di * P, img = g_first / P + di;
    o_at[bj] = (uint32_t)(img * args.M * PQ + p * Q + q);
    const uint32_t at = rows_window(img * Hp + p * stride - R0, q * stride - pad + XO, row_pitch, ES);
    b_at[bj] = at & ~3u;
    b_odd[bj] = at & 2u;
  }

  // ---- one stage: two chunks (one per lane group) and MBLK x NBLK MFMAs per step, the next step's reads in flight
  u32x4 af[2][C::MBLK];
  uint32_t bd[2][C::NBLK][5];
  auto compute = [&](int ch) {
    const int nch = ch * R * SC;
    const int steps = (nch + 1) >> 1;
    RowsWalk<ONE_CHUNK> walk;                            // where the lane's chunk of the next step lies
    auto advance = [&]() { walk.advance(R, SC, row_pitch, chan_pitch); };
    const uint32_t last_off = walk.last(ch, R, SC, row_pitch, chan_pitch);
    if (fgrp) advance();
    int valid[2] = {S, S};                               // elements of the filter row in the lane's chunk
    GENSOR_LDS char* arow = abase + (wave_m * C::WM + frow) * a_pitch + fgrp * 16;
    auto read = [&](int buf, int step) {
      if constexpr (!ONE_CHUNK) valid[buf] = S - walk.sc * EPC;
#pragma unroll
      for (int bi = 0; bi < C::MBLK; ++bi) af[buf][bi] = *(GENSOR_LDS u32x4*)(arow + bi * MB * a_pitch + step * 32);
      const uint32_t off = walk.at(last_off);
#pragma unroll
      for (int bj = 0; bj < C::NBLK; ++bj) {
        GENSOR_LDS uint32_t* src = (GENSOR_LDS uint32_t*)(pbase + b_at[bj] + off);
#pragma unroll
        for (int e = 0; e < (ES == 2 ? 5 : 4); ++e) bd[buf][bj][e] = src[e];
      }
      advance();
      advance();
    };
    // the last step's second chunk may be the zero one that makes the count even: its window is cleared, too (`last`)
    auto mma = [&](int buf, auto last_tag) {
      constexpr bool last = decltype(last_tag)::value;
      const int n = last && 2 * steps - 2 + fgrp >= nch ? 0 : valid[buf];
      u32x4 bf[C::NBLK];
#pragma unroll
      for (int bj = 0; bj < C::NBLK; ++bj)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (ES == 4) bf[bj][e] = bd[buf][bj][e] & dword_mask(n, e);
          else bf[bj][e] = __builtin_amdgcn_alignbyte(bd[buf][bj][e + 1], bd[buf][bj][e], b_odd[bj]) & dword_mask(n, e);
        }
#pragma unroll
      for (int bi = 0; bi < C::MBLK; ++bi)
#pragma unroll
        for (int bj = 0; bj < C::NBLK; ++bj) MF::run(af[buf][bi], bf[bj], acc[bi][bj]);
    };
    read(0, 0);
    int step = 0;
    for (; step + 2 < steps; step += 2) {
      read(1, step + 1);
      mma(0, std::false_type{});
      read(0, step + 2);
      mma(1, std::false_type{});
    }
    if (step + 1 < steps) {
      read(1, step + 1);
      mma(0, std::false_type{});
      mma(1, std::true_type{});
    } else {
      mma(0, std::true_type{});
    }
  };

  __syncthreads();                       // the zero fill before the first rows
  for (int c0 = 0; c0 < Cc; c0 += stage_ch) {
    if (c0) __syncthreads();             // everyone has read the stage before
    for (int b = 0; b < batches; ++b) stage(c0, b);
    __syncthreads();
    if (!idle) compute(min(stage_ch, Cc - c0));
  }

  // ---- epilogue: O[img][filter][p][q], written through (the output is most of the traffic)
  if (idle) return;
  typedef typename C::OutT OutT;
  constexpr int OS = ElemSize<OutT>::value;
  const __amdgpu_buffer_rsrc_t rs_out = __builtin_amdgcn_make_buffer_rsrc((void*)args.C, 0, (uint32_t)args.cOutBytes, RSRC_FLAGS);
  constexpr int WRITE_THROUGH = 16;
  const uint32_t row_bytes = (uint32_t)(PQ * OS);
  auto store = [&](auto whole_tag) {                     // whole: every filter of the tile exists
    constexpr bool whole = decltype(whole_tag)::value;
    const int row0 = m0 + wave_m * C::WM + 4 * fgrp;
#pragma unroll
    for (int bj = 0; bj < C::NBLK; ++bj) {
      // (an offset at or above OOB stays out of range when row offsets below 2^31 are added)
      const uint32_t first = n0 + wave_n * C::WN + bj * MB + frow < n_end ? o_at[bj] * OS + (uint32_t)row0 * row_bytes : OOB;
#pragma unroll
      for (int bi = 0; bi < C::MBLK; ++bi)
#pragma unroll
        for (int v = 0; v < MF::NACC; ++v) {
          const int r = bi * MB + 8 * (v / 4) + (v % 4);
          uint32_t off = first + (uint32_t)r * row_bytes;
          if constexpr (!whole) off = row0 + r < args.M ? off : OOB;
          if constexpr (OS == 4) {
            __builtin_amdgcn_raw_buffer_store_b32(as_u32(acc[bi][bj][v]), rs_out, off, 0, WRITE_THROUGH);
          } else {
            uint16_t bits;
            store_out<OutT>(&bits, 0, acc[bi][bj][v]);
            __builtin_amdgcn_raw_buffer_store_b16(bits, rs_out, off, 0, WRITE_THROUGH);
          }
        }
    }
  };
  if (m0 + BM <= args.M) store(std::true_type{});
  else store(std::false_type{});
}

}  // namespace gensor
