// Scheduled dense-contraction kernel for gfx950 (CDNA4): one template covers GEMM, batched
// matmul and implicit-GEMM convolution.  Every template parameter is a schedule primitive
// of the construction graph (Section IV-A of the paper: per-level tiles, caching, virtual
// threads; Table I: unroll, vectorise):
//
//   BM,BN,BK   T_2  workgroup tile, staged in LDS                ("cache" primitive)
//   WM,WN      T_1  wavefront tile, fp32 accumulators in registers
//   MB         MFMA block edge (32: 32x32 blocks, 16: 16x16 blocks); fixes the MFMA k depth
//   VM,VN      virtual threads (setVThread, Eq. 3): the rows that one quarter wave reads together
//              from the LDS tile of the m (A) or n (B) operand are interleaved over V bank phases;
//              V = 1 is the plain layout, whose fragment reads conflict ceil(x / W) ways
//   STAGES     LDS buffers (1: single buffer, 2: double buffer, 3 and more: a ring that keeps STAGES-1
//              k tiles in flight; direct staging only)
//   VEC        operands start every row on a 16-byte boundary and rows are whole vectors (true), or lie
//              anywhere on element boundaries with any extents (false)
//   DIRECT     K-contiguous operands go global->LDS without passing through registers
//
// Operand sources.  A (the m x k operand) is k-contiguous, A[m][k] (A_KC), or m-contiguous, A stored
// [k][m] (A_MC, "transA": staged and read exactly like an n-contiguous B).  B is
//   KC   k-contiguous,  B stored [n][k]   (column-major B / "transB")
//   NC   n-contiguous,  B stored [k][n]   (row-major B)
//   CONV n = (image, out row, out col), k = (channel, filter row, filter col): element
//        (k, n) is gathered from the NCHW input, zero outside the image; m = filter.
//
// LDS layouts.  k-contiguous tiles are [rows][BK] in 16-byte chunks; chunk c of row r sits
// at chunk c ^ ((r / rows_per_256B) % V).  The 16 rows that a quarter wave's b128 fragment read
// touches span x = 16 * min(row bytes, 256) bytes, i.e. ceil(x / (V * 256)) of them share each
// bank: with V = chunks per row the read hits 64 distinct banks.  n-contiguous tiles are
// [BK][BN + pad]; their V is the number of k rows that the pad (or, direct-staged, an XOR of the
// column bytes) spreads over different banks: 4 rows are read together by a transposing 16-bit
// read (pad 0 / 32 / 64 bytes for V = 1 / 2 / 4), 2 by a 32-bit one (pad 0 / 32).
//
// MFMA operand convention (per lane l of a 64-wide wave):
//   32x32 blocks: row/col = l % 32, holds the 16-byte chunk  2*kstep + l/32  of that row
//   16x16 blocks: row/col = l % 16, holds the 16-byte chunk  4*kstep + l/16  of that row
// For 16-bit types a chunk is 8 consecutive k and feeds one MFMA; for fp32 a chunk is 4
// consecutive k and feeds 4 MFMAs (element t of the chunk at step t).  The order in which k
// is consumed differs from memory order, identically for both operands.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <stdint.h>

namespace gensor {

// B_NCS2: n-contiguous B whose column n = p*Q + q is read at (2p)*W + 2q of a plane of H*W elements
// (= ldb): the input of a pointwise convolution with stride 2, sampled while it is fetched.
enum BSrc { B_KC = 0, B_NC = 1, B_CONV = 2, B_NCS2 = 3 };
enum ASrc { A_KC = 0, A_MC = 1 };

struct KernelArgs {
  const void* A;
  const void* B;
  void* C;
  int32_t M, N, K;                 // GEMM-view extents
  int64_t lda, ldb, ldc;           // elements
  int64_t strideA, strideB, strideC;
  float alpha, beta;
  int32_t through;                 // C is stored write-through (beside beta only with fp32 output)
  int32_t paired;                  // 16-bit C without beta whose columns 2j and 2j + 1 are one aligned dword
  int32_t lds_stages;              // LDS stages a launch allocates at most (its k tiles, where fewer than the instance's)
  int32_t narrow;                  // tiles of 192 instead of 256 columns (instances whose wave groups alternate; the launch selects them)
  int32_t tiles_m, tiles_n, batch;
  int32_t panel;                   // tile rows per panel in the workgroup->tile map
  int64_t ahead_a, ahead_b;        // bytes of the next batch's A and B that this batch's workgroups read ahead (0: none)
  // split-k: workgroups [0, whole) compute one whole tile each; the tiles behind them are computed by
  // `split` workgroups each, every one over its own range of k tiles (split == 1: whole == all tiles)
  int32_t split, whole;
  float* partials;                 // [tile - whole][split][BM * BN] fp32, lane-major inside a slot
  // convolution geometry (B_CONV only)
  int32_t cC, cH, cW, cR, cS, cP, cQ, cStride, cPad;
  // patch-staged convolution only: images, LDS plan and tensor sizes in bytes (each < 2^31)
  int32_t cN, cApitch, cPatchRows, cStageBytes;
  int32_t cRowPitch, cStageCh;     // row-staged convolution only: bytes of an input row in LDS, channels per stage
  uint32_t cRec[7];                // ... and ceil(2^32 / d) (0 for d = 1) of what its kernel divides by
  int32_t cTilePx;                 // output pixels per workgroup (at most BN; whole output rows when they are shorter than BN)
  int64_t cInBytes, cWBytes, cOutBytes;
};

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

#define GENSOR_LDS __attribute__((address_space(3)))

struct f16_t { typedef _Float16 native; };
struct bf16_t { typedef __bf16 native; };
struct f32_t { typedef float native; };

template <typename T> struct ElemSize { static constexpr int value = 2; };
template <> struct ElemSize<f32_t> { static constexpr int value = 4; };

// ---------------------------------------------------------------- scalar conversions
template <typename T> __device__ inline float to_float(const void* p, int64_t i);
template <> __device__ inline float to_float<f32_t>(const void* p, int64_t i) { return ((const float*)p)[i]; }
template <> __device__ inline float to_float<f16_t>(const void* p, int64_t i) { return (float)((const _Float16*)p)[i]; }
template <> __device__ inline float to_float<bf16_t>(const void* p, int64_t i) {
  return __builtin_bit_cast(float, ((uint32_t)((const uint16_t*)p)[i]) << 16);
}
template <typename T> __device__ inline void store_out(void* p, int64_t i, float v);
template <> __device__ inline void store_out<f32_t>(void* p, int64_t i, float v) { ((float*)p)[i] = v; }
template <> __device__ inline void store_out<f16_t>(void* p, int64_t i, float v) { ((_Float16*)p)[i] = (_Float16)v; }
template <> __device__ inline void store_out<bf16_t>(void* p, int64_t i, float v) {
  uint32_t u = __builtin_bit_cast(uint32_t, v);                 // round to nearest even
  uint32_t r = (u & 0x7fffffffu) > 0x7f800000u ? 0x7fc0u : ((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
  ((uint16_t*)p)[i] = (uint16_t)r;
}

// two values rounded to nearest even, the first in the low half
template <typename T> __device__ inline uint32_t pack_out(float lo, float hi) {
  typedef typename T::native pair_t __attribute__((ext_vector_type(2)));
  const pair_t p = {(typename T::native)lo, (typename T::native)hi};
  return __builtin_bit_cast(uint32_t, p);
}

// 16 bytes a lane to lds + 16 * lane.  (The host's pass knows no 16-byte form of the builtin, and would drop the kernel.)
__device__ inline void load_to_lds(__amdgpu_buffer_rsrc_t r, GENSOR_LDS char* lds, uint32_t offset) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (GENSOR_LDS void*)lds, 16, offset, 0, 0, 0);
#endif
}

// ---------------------------------------------------------------- MFMA wrappers
// (the bits travel through a by-value argument: a bit cast applied directly to a vector
// element expression reads element 0 whatever the index)
__device__ inline float as_f32(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ inline uint32_t as_u32(float f) { return __builtin_bit_cast(uint32_t, f); }

template <typename T, int MB> struct Mfma;
template <> struct Mfma<f16_t, 32> {
  typedef f32x16 Acc;
  static constexpr int NACC = 16;
  __device__ static inline void run(const u32x4& a, const u32x4& b, Acc& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mfma<f16_t, 16> {
  typedef f32x4 Acc;
  static constexpr int NACC = 4;
  __device__ static inline void run(const u32x4& a, const u32x4& b, Acc& c) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mfma<bf16_t, 32> {
  typedef f32x16 Acc;
  static constexpr int NACC = 16;
  __device__ static inline void run(const u32x4& a, const u32x4& b, Acc& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mfma<bf16_t, 16> {
  typedef f32x4 Acc;
  static constexpr int NACC = 4;
  __device__ static inline void run(const u32x4& a, const u32x4& b, Acc& c) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mfma<f32_t, 32> {   // true fp32 multiply-add: 32x32x2 per step, 4 steps per chunk
  typedef f32x16 Acc;
  static constexpr int NACC = 16;
  __device__ static inline void run(const u32x4& a, const u32x4& b, Acc& c) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(as_f32(a[t]), as_f32(b[t]), c, 0, 0, 0);
  }
};
template <> struct Mfma<f32_t, 16> {   // 16x16x4 per step
  typedef f32x4 Acc;
  static constexpr int NACC = 4;
  __device__ static inline void run(const u32x4& a, const u32x4& b, Acc& c) {
#pragma unroll
    for (int t = 0; t < 4; ++t) step(a, b, t, c);
  }
  __device__ static inline void step(const u32x4& a, const u32x4& b, int t, Acc& c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(as_f32(a[t]), as_f32(b[t]), c, 0, 0, 0);
  }
};

// ---------------------------------------------------------------- schedule -> constants
template <typename T_, typename OutT_, int BM_, int BN_, int BK_, int WM_, int WN_, int MB_, int VM_, int VN_,
          int BSRC_, bool VEC_, int STAGES_, bool DIRECT_, int ASRC_ = A_KC>
struct Cfg {
  typedef T_ T;
  typedef OutT_ OutT;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, MB = MB_, VM = VM_, VN = VN_;
  static constexpr int BSRC = BSRC_, STAGES = STAGES_, ASRC = ASRC_;
  static constexpr bool VEC = VEC_, DIRECT = DIRECT_;
  static constexpr int ES = ElemSize<T>::value;
  static constexpr int EPC = 16 / ES;                        // elements per 16-byte chunk
  static constexpr int WAVES_M = BM / WM, WAVES_N = BN / WN, WAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = WAVES * 64;
  static constexpr int MBLK = WM / MB, NBLK = WN / MB;       // MFMA blocks per wave tile
  static constexpr int LANE_GROUPS = 64 / MB;                // 2 (32x32) or 4 (16x16)
  static constexpr int KG = LANE_GROUPS * EPC;               // k consumed per fragment read
  static constexpr int KSTEPS = BK / KG;                     // the "unroll" of the schedule
  // k-contiguous LDS tile: [rows][BK], 16-byte chunks, xor swizzle
  static constexpr int PITCH_K = BK * ES;                    // bytes per row
  static constexpr int CPR = PITCH_K / 16;                   // chunks per row
  static constexpr int RPP = (PITCH_K >= 256) ? 1 : 256 / PITCH_K;   // rows per 256-byte bank period
  // n-contiguous LDS tile: [BK][BN] + pad
  // (direct staging deposits whole 1 KB runs, so there the rows are unpadded and 32-byte
  // column segments are XOR-swizzled with the k row instead)
  static constexpr bool NC_DIRECT = DIRECT_ && BSRC_ == B_NC;
  static constexpr bool MC_DIRECT = DIRECT_ && ASRC_ == A_MC;
  static constexpr int V_MAX_K = CPR;                        // deepest interleave of a k-contiguous tile
  static constexpr int V_MAX_N = (ES == 2) ? 4 : 2;          // ... of an n-contiguous tile
  // the pad puts consecutive k rows 64 bytes (V = 4) or 32 bytes (V = 2) apart modulo the 256 bytes of all banks
  static constexpr int PAD_T = (VN >= 4) ? 64 : 32;
  static constexpr int PAD_N = (VN == 1) ? 0 : (PAD_T + 2 * PAD_T - (BN * ES) % (2 * PAD_T)) % (2 * PAD_T);
  static constexpr int PITCH_N = NC_DIRECT ? BN * ES : BN * ES + PAD_N;
  // m-contiguous A tile: [BK][BM] + pad, the same rule
  static constexpr int PAD_TM = (VM >= 4) ? 64 : 32;
  static constexpr int PAD_M = (VM == 1) ? 0 : (PAD_TM + 2 * PAD_TM - (BM * ES) % (2 * PAD_TM)) % (2 * PAD_TM);
  static constexpr int PITCH_M = MC_DIRECT ? BM * ES : BM * ES + PAD_M;
  static constexpr int A_BYTES = (ASRC == A_KC) ? BM * PITCH_K : BK * PITCH_M;
  static constexpr int B_BYTES = (BSRC == B_KC) ? BN * PITCH_K : BK * PITCH_N;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  // Two groups of four waves that take turns at reading and multiplying (the loop says how); B has a third stage.
  static constexpr bool ALTERNATE = DIRECT_ && STAGES_ == 2 && MB_ == 16 && ES == 2 && BM_ == 256 && BK_ == 64 &&
                                    ((BN_ == 256 && WM_ == 128 && WN_ == 64) || (BN_ == 192 && WM_ == 64 && WN_ == 96));
  static constexpr bool HAS_NARROW = ALTERNATE && BN_ == 256;
  // Rings of 16x16 blocks: the same products for less power than 32x32 ones (beside the alternating tiles' loop), and they take any K.
  // 32x32 -> 16x16, us: 2048^3 f16 22.5 -> 20.4, 512 x 512 x 32768 in 16 parts 28.7 -> 26.7, 256x128 tiles 4096 x 2048 x 2048 36.4 ->
  // 33.1, with 16-bit output 32.9 -> 30.3, 768 x 3072 x 8192 transA in three parts 50.8 -> 48.2.  (On all-zero operands they are level.)
  static constexpr bool RING_16 = DIRECT_ && STAGES_ > 2 && MB_ == 16;
  static constexpr int LDS_BYTES = STAGE_BYTES * STAGES + (ALTERNATE ? B_BYTES : 0);
  static constexpr int A_CHUNKS = (ASRC == A_KC) ? BM * CPR : BK * (BM * ES / 16);
  static constexpr int B_CHUNKS = (BSRC == B_KC) ? BN * CPR : BK * (BN * ES / 16);
  static constexpr int A_LOADS = (A_CHUNKS + THREADS - 1) / THREADS;
  static constexpr int B_LOADS = (B_CHUNKS + THREADS - 1) / THREADS;
  // Register-staged double buffer: two register sets, i.e. two k tiles of loads in flight, where they fit beside the
  // accumulators, the fragments and the addresses into the 256 registers of a lane that two waves per SIMD leave
  // (a set more than that would halve the resident waves).  16x16 blocks compile to about half as many fragment registers again as the two
  // steps' (128x128x64 tiles: 264-284 registers with two sets, one workgroup per CU instead of two, 8192 x 4096 x 512
  // 60 -> 72 us, 16384 x 2048 x 192 33 -> 44).
  static constexpr int STAGE_REGS = 4 * (A_LOADS + B_LOADS * (BSRC_ == B_NCS2 ? 2 : 1));
  static constexpr int OTHER_REGS = WM_ * WN_ / 64 + (MB_ == 16 ? 12 : 8) * (MBLK + NBLK) + 2 * (A_LOADS + B_LOADS) + 24;
  static constexpr int RSETS = (!DIRECT_ && STAGES_ == 2 && KSTEPS % 2 == 0 && BSRC_ != B_CONV && 2 * STAGE_REGS + OTHER_REGS <= 256) ? 2 : 1;
  // Small tiles of deep k tiles stand where parts of split tiles stood, whose shorter chains of sums lose less to rounding: they keep as
  // many sums per output as such a split had parts, an eighth of the products each (16-bit: one k step of every other k tile), added up at the end (512^3 fp32 6.14 us, 5.97 with one
  // chain and 6.28 with sixteen; compiled with the accumulators in plain registers, between which and the others they were copied in every k
  // tile: 7.2).  In one chain an fp32 product of depth 600 was 3.7e-7 from 64 bits, where its
  // split in eight had been 1.5e-7; over 85 drawn products whose schedule changed the distance is now 0.77 of what it was (geometric mean).
  static constexpr int CHAINS = DIRECT_ || MB_ != 16 || BK_ * ES != 256 || MBLK * NBLK > 2 ? 1 : 8;
  // More sums per output in launches of a deep k, where tiles that others once took in (more) parts are whole (launch_instance; at 16-bit output
  // its rounding is a thousand times larger).  Without them, distance from 64 bits with the parts and with the whole: 589 x 1163 x 1643
  // f16 any-alignment, four parts 1.37e-7, one tile 2.59e-7 (four sums 1.36e-7); 3072 x 768 x 7352 f16 transA 2.28e-7, 3.16e-7 (two 2.27e-7);
  // 1792 x 1152 x 2176 bf16 2.60e-7 (four 1.23e-7).  For it 64x32 waves of the rings have registers for four, 64x64 ones for two, and the
  // any-alignment tile needs 150-160 instead of 96-104.
  static constexpr bool LOOSE_64 = !DIRECT_ && !VEC_ && BN_ == 64 && RSETS == 2 && (ES == 2 ? (BM_ == 64 || BM_ == 128) && BK_ == 64 : BM_ == 64 && BK_ == 32);
  static constexpr int DEEP_CHAINS = ElemSize<OutT_>::value != 4 ? CHAINS : RING_16 ? (BM_ * BN_ == 128 * 128 ? 4 : 2) : LOOSE_64 ? (ES == 4 ? 8 : BM_ == 64 ? 4 : 2) : CHAINS;
  // the tile that store-bound batches of a shallow k end in also exists with the next batch read ahead
  static constexpr bool HAS_AHEAD = VEC_ && DIRECT_ && STAGES_ == 2 && ES == 2 && ElemSize<OutT_>::value == 4 && BM_ == 128 && BN_ == 128 && WAVES == 8;
  static_assert(BM % WM == 0 && BN % WN == 0, "wave tile must divide workgroup tile");
  static_assert(WM % MB == 0 && WN % MB == 0, "wave tiles are whole MFMA blocks");
  static_assert(VM >= 1 && (VM & (VM - 1)) == 0 && VM <= (ASRC == A_KC ? V_MAX_K : V_MAX_N), "V of the m operand: a power of two up to the chunks per row");
  static_assert(ASRC == A_KC || (BSRC != B_CONV && BSRC != B_NCS2), "an m-contiguous A is for GEMM only");
  static_assert(!MC_DIRECT || (ES == 2 && BM * ES / 16 >= 16 && A_CHUNKS % THREADS == 0), "its direct staging deposits whole waves of swizzled rows of at least 16 chunks");
  static_assert(VN >= 1 && (VN & (VN - 1)) == 0 && VN <= (BSRC == B_KC ? V_MAX_K : V_MAX_N), "V of the n operand");
  static_assert(BK % KG == 0, "BK must be a multiple of the fragment k extent");
  static_assert(MB == 32 || MB == 16, "MFMA block edge");
  static_assert(WAVES >= 1 && WAVES <= 16, "waves per workgroup");
  static_assert(!DIRECT || (VEC && (BSRC == B_KC || (BSRC == B_NC && BN * ES / 16 >= 16))),
                "direct-to-LDS needs vector loads; an n-contiguous B needs rows of at least 16 chunks for its swizzle");
  static_assert(!NC_DIRECT || (B_CHUNKS % THREADS == 0), "direct staging deposits whole waves");
  static_assert(BSRC != B_NCS2 || VEC, "the sampled source exists only with aligned vector loads");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS capacity");
  static_assert(STAGES <= 2 || (DIRECT && VEC && (BSRC == B_KC || BSRC == B_NC) && KSTEPS % 2 == 0),
                "rings of three and more stages are filled by direct loads");
  static_assert(STAGES <= 2 || (A_LOADS + B_LOADS) * (STAGES - 2) <= 63, "the load counter holds 63");
};

// The 192-column form of an instance whose wave groups alternate: three quarters of the work a tile for the shapes whose 256-column
// tiles end in a partly filled round (8192 x 3072 x 768: 384 tiles of 256 columns are one and a half rounds, 512 of 192 two full ones;
// 42.2 -> 38.8 us, 2880 x 3648 x 2048 50.2 -> 45.1, 3264 x 2560 x 3264 64.5 -> 60.0).  On all-zero operands a k tile
// takes 1648 cycles of 2.4 GHz with a k-contiguous B and 1960 with a row-major one, beside 1536 of products (256 columns: 2122 and
// 2168 beside 2048); on uniform ones, under the power limit, 2510 and 2758 (3085 and 3252).
template <typename C>
using NarrowCfg = Cfg<typename C::T, typename C::OutT, 256, 192, 64, 64, 96, 16, C::VM, C::VN, C::BSRC, true, 2, true, C::ASRC>;

__device__ inline int swizzled_chunk(int row, int chunk, int rpp, int v) { return chunk ^ ((row / rpp) % v); }
// Byte XOR applied inside an unpadded n-contiguous row of k row `krow`: of the four rows a
// 16-lane group of a transposing read touches, v land in different 64-byte bank groups (v = 4:
// all of them), and with v = 4 rows 8 apart (the two groups of a 16x16-block read) in
// different 32-byte halves.
__device__ inline int nc_swizzle(int krow, int v) { return ((krow & (v - 1)) << 6) ^ (v >= 4 ? (((krow >> 3) & 1) << 5) : 0); }

template <int N, int I = 0, typename F>
__device__ inline __attribute__((always_inline)) void static_for(F&& f) {      // f(integral_constant<int, 0 .. N-1>)
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Workgroup ids are dealt round-robin to the 8 XCDs.  Number `id` of `count` so that each XCD holds a contiguous range (the
// first count % 8 of them one more).  Counts that are not a multiple of 8 were left scattered once, so that every XCD fetched all
// operands: 39 x 669 x 669 x 64 fp16 18.0 -> 15.4 us, 91 x 364 x 364 x 128 bf16 18.6 -> 15.7, split 672 x 344 x 16832 in parts of
// other counts 1.2 times faster; a pointwise layer of 27 x 128 x 28 x 28 -> 416 12.9 -> 10.5.
__device__ inline int xcd_contiguous(int id, int count) {
  const int xcd = id & 7;
  return xcd * (count >> 3) + min(xcd, count & 7) + (id >> 3);
}

// Do k tiles kt .. kt + n - 1 of bk rows, and `beyond` more rows, lie inside K?  (Nothing here exceeds K + n * bk in magnitude as long as
// tile kt starts inside it: K may be anything up to INT32_MAX.)
__host__ __device__ constexpr bool tiles_inside(int kt, int n, int bk, int beyond, int K) { return kt * bk <= K - (n * bk + beyond); }

// tile number inside a batch -> tile coordinates: panels of `panel` tile rows, walked column by column
__device__ inline void tile_of(const KernelArgs& args, int t, int& tile_m, int& tile_n) {
  const int panel = args.panel;
  const int per_panel = panel * args.tiles_n;
  const int pi = t / per_panel;
  const int rows_here = min(panel, args.tiles_m - pi * panel);
  const int r = t - pi * per_panel;
  tile_m = pi * panel + r % rows_here;
  tile_n = r / rows_here;
}

// ---------------------------------------------------------------- the kernel
// SPLIT: the launch has split tiles (KernelArgs::split > 1); without it the kernel knows at compile time
// that every workgroup owns a whole tile.  AHEAD: workgroups read the next batch's operands ahead (KernelArgs::ahead_a;
// carrying the unused load through every launch cost the small batched ones 1-2 %).  MORE_SUMS: Cfg::DEEP_CHAINS.
template <typename C, bool SPLIT = false, bool AHEAD = false, bool MORE_SUMS = false>
__global__ __launch_bounds__(C::THREADS) void contraction_kernel(const KernelArgs args) {
  typedef typename C::T T;
  typedef Mfma<T, C::MB> MF;
  typedef typename MF::Acc Acc;
  constexpr int ES = C::ES, EPC = C::EPC, BM = C::BM, BN = C::BN, BK = C::BK, MB = C::MB;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  GENSOR_LDS char* lds = (GENSOR_LDS char*)smem;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
  const int wave_m = wave / C::WAVES_N;
  const int wave_n = wave % C::WAVES_N;

  // ---- workgroup -> (batch, tile_m, tile_n).  Consecutive workgroup ids are dealt
  // round-robin to the 8 XCDs; give each XCD a contiguous range of tiles, and walk tiles
  // in panels of `panel` tile rows so that the tiles resident on one XCD share operand
  // slabs in that XCD's L2.
  const int tiles_per_batch = args.tiles_m * args.tiles_n;
  const int total = tiles_per_batch * args.batch;
  int wg = blockIdx.x;
  int kpart = 0, kparts = 1;                // this workgroup's share of a split tile
  if constexpr (!SPLIT) {
    wg = xcd_contiguous(wg, total);
  } else if (wg < args.whole) {
    wg = xcd_contiguous(wg, args.whole);
  } else {
    // the split tiles come last in launch order, part by part: an XCD then holds neighbouring tiles over one range of
    // k and its L2 fetches each operand's range once for all of them.  Tile by tile it fetched the slabs of its few tiles
    // over the whole of k: 512 x 512 x 32768 in 16 parts read its operands three times over, 38.7 against 29-30 us.
    kparts = args.split;
    const int tiles = total - args.whole, units = tiles * kparts;
    const int u = xcd_contiguous(wg - args.whole, units);
    kpart = u / tiles;
    wg = args.whole + u - kpart * tiles;
  }
  const int bidx = wg / tiles_per_batch;
  int tile_m, tile_n;
  tile_of(args, wg - bidx * tiles_per_batch, tile_m, tile_n);
  const int m0 = tile_m * BM;
  const int n0 = tile_n * BN;

  // k range of this workgroup: the whole of K, or k tiles [kpart * nk / kparts, (kpart + 1) * nk / kparts) of a split
  // tile.  The operand bases move to the first k of the range and Kx is its length, so everything below
  // sees a shorter contraction.
  int Kx = args.K;
  int64_t k_first = 0;
  if (SPLIT && kparts > 1) {
    const int nk_all = (args.K + BK - 1) / BK;
    const int kt0 = kpart * nk_all / kparts, kt1 = (kpart + 1) * nk_all / kparts;
    k_first = (int64_t)kt0 * BK;
    Kx = min(args.K, kt1 * BK) - kt0 * BK;
  }
  const char* Ab = (const char*)args.A + ((int64_t)bidx * args.strideA + (C::ASRC == A_KC ? k_first : k_first * args.lda)) * ES;
  const char* Bb = (const char*)args.B + ((int64_t)bidx * args.strideB + (C::BSRC == B_KC ? k_first : k_first * args.ldb)) * ES;

  // ---- accumulators
  Acc acc[C::MBLK][C::NBLK];
#pragma unroll
  for (int i = 0; i < C::MBLK; ++i)
#pragma unroll
    for (int j = 0; j < C::NBLK; ++j)
#pragma unroll
      for (int v = 0; v < MF::NACC; ++v) acc[i][j][v] = 0.f;
  constexpr int CHAINS = MORE_SUMS ? C::DEEP_CHAINS : C::CHAINS;
  Acc more_acc[CHAINS > 1 ? CHAINS - 1 : 1][C::MBLK][C::NBLK];       // ... of the further chains of a block
  auto chain = [&](int n, int i, int j) -> Acc& { return n == 0 ? acc[i][j] : more_acc[n - 1][i][j]; };
  if constexpr (CHAINS > 1) {
#pragma unroll
    for (int n = 1; n < CHAINS; ++n)
#pragma unroll
      for (int i = 0; i < C::MBLK; ++i)
#pragma unroll
        for (int j = 0; j < C::NBLK; ++j)
#pragma unroll
          for (int v = 0; v < MF::NACC; ++v) chain(n, i, j)[v] = 0.f;
  }

  // ---- buffer resources.  Each operand is addressed through a buffer descriptor whose
  // base is this workgroup's first row (or column) at the current k tile and whose extent
  // ends with the matrix: out-of-range lanes read zero (or are dropped on store) in
  // hardware, so the loop body has no branches.  Offsets inside a tile stay below 2^31 (the
  // host checks BM * lda, BN * ldb or BK * ldb, and BM * ldc).
  constexpr uint32_t RSRC_FLAGS = 0x00020000u;
  constexpr uint32_t OOB = 0x80000000u;      // beyond every descriptor (extents are clamped below 2^31)
  auto clamp_records = [](int64_t bytes) -> uint32_t {
    return bytes <= 0 ? 0u : (bytes > 0x7fffffffll ? 0x7fffffffu : (uint32_t)bytes);
  };
  const int rows_valid = min(BM, args.M - m0);
  const int cols_valid = min(BN, args.N - n0);
  const char* a_tile = (C::ASRC == A_KC) ? Ab + (int64_t)m0 * args.lda * ES : Ab + (int64_t)m0 * ES;
  const char* b_tile = (C::BSRC == B_KC) ? Bb + (int64_t)n0 * args.ldb * ES : (C::BSRC == B_NCS2 ? Bb : Bb + (int64_t)n0 * ES);
  // Operands without VEC start anywhere: the descriptor begins at the 16-byte granule that holds the tile's first
  // element (`skew` bytes before it) and ends on a dword boundary, so that it covers every dword that holds an
  // element; a granule or dword that holds one lies in the element's own page.
  auto loose_rsrc = [&](const char* first, int64_t bytes, uint32_t& skew) {
    skew = (uint32_t)((uintptr_t)first & 15u);
    return __builtin_amdgcn_make_buffer_rsrc((void*)(first - skew), 0, bytes <= 0 ? 0u : clamp_records((bytes + skew + 3) & ~3ll), RSRC_FLAGS);
  };
  auto rsrc_a = [&](int k0) {
    if constexpr (C::ASRC == A_KC)
      return __builtin_amdgcn_make_buffer_rsrc((void*)(a_tile + (int64_t)k0 * ES), 0,
          clamp_records(((int64_t)(rows_valid - 1) * args.lda + (Kx - k0)) * ES), RSRC_FLAGS);
    else      // k rows beyond K fall out of range; rows of the tile beyond M read what follows them and are never stored
      return __builtin_amdgcn_make_buffer_rsrc((void*)(a_tile + (int64_t)k0 * args.lda * ES), 0,
          clamp_records(((int64_t)(Kx - k0 - 1) * args.lda + (args.M - m0)) * ES), RSRC_FLAGS);
  };
  auto rsrc_b = [&](int k0) {
    if constexpr (C::BSRC == B_KC)
      return __builtin_amdgcn_make_buffer_rsrc((void*)(b_tile + (int64_t)k0 * ES), 0,
          clamp_records(((int64_t)(cols_valid - 1) * args.ldb + (Kx - k0)) * ES), RSRC_FLAGS);
    else if constexpr (C::BSRC == B_NCS2)
      return __builtin_amdgcn_make_buffer_rsrc((void*)(b_tile + (int64_t)k0 * args.ldb * ES), 0,
          clamp_records((int64_t)(Kx - k0) * args.ldb * ES), RSRC_FLAGS);
    else
      return __builtin_amdgcn_make_buffer_rsrc((void*)(b_tile + (int64_t)k0 * args.ldb * ES), 0,
          clamp_records(((int64_t)(Kx - k0 - 1) * args.ldb + (args.N - n0)) * ES), RSRC_FLAGS);
  };

  // ---- who loads what.  A thread owns LDS chunk slots q = tid + i*THREADS of a
  // k-contiguous tile (slot q = row q/CPR, physical chunk q%CPR) and fetches the logical
  // chunk that the swizzle maps there; the same ownership serves the register-staged and
  // the direct path (a direct load deposits lane l's 16 bytes at slot base + l).
  constexpr bool LOOSE_A = !C::VEC;
  constexpr bool GATHER_B = C::BSRC == B_CONV;
  constexpr bool LOOSE_B = !C::VEC && !GATHER_B;
  uint32_t a_voff[C::A_LOADS], a_kch[C::A_LOADS];
#pragma unroll
  for (int i = 0; i < C::A_LOADS; ++i) {
    const int q = tid + i * C::THREADS;
    if constexpr (C::ASRC == A_KC) {
      const int row = q / C::CPR, ch = swizzled_chunk(row, q % C::CPR, C::RPP, C::VM);
      a_voff[i] = (uint32_t)((row * (int)args.lda + ch * EPC) * ES);
      a_kch[i] = ch * EPC;
    } else {
      constexpr int CPRM = BM * ES / 16;
      int ch = q % CPRM;
      if constexpr (C::MC_DIRECT) ch ^= nc_swizzle(q / CPRM, C::VM) >> 4;
      a_voff[i] = (uint32_t)(((q / CPRM) * (int)args.lda + ch * EPC) * ES);
      a_kch[i] = q / CPRM;
    }
  }
  uint32_t b_voff[C::B_LOADS], b_kch[C::B_LOADS];
  uint32_t b_voff2[C::BSRC == B_NCS2 ? C::B_LOADS : 1];      // second half of a sampled chunk
#pragma unroll
  for (int i = 0; i < C::B_LOADS; ++i) {
    const int q = tid + i * C::THREADS;
    if constexpr (C::BSRC == B_KC) {
      const int row = q / C::CPR, ch = swizzled_chunk(row, q % C::CPR, C::RPP, C::VN);
      b_voff[i] = (uint32_t)((row * (int)args.ldb + ch * EPC) * ES);
      b_kch[i] = ch * EPC;
    } else if constexpr (C::BSRC == B_NCS2) {
      // chunk = EPC consecutive columns = two halves of EPC/2 columns, each inside one output
      // row (Q is a multiple of EPC/2) and so one 16-byte run of the input row it samples
      constexpr int CPRN = BN * ES / 16;
      const int krow = q / CPRN, ch = q % CPRN;
      const int nA = n0 + ch * EPC, nB = nA + EPC / 2;
      const int pA = nA / args.cQ, pB = nB / args.cQ;
      const int sA = (2 * pA) * args.cW + 2 * (nA - pA * args.cQ), sB = (2 * pB) * args.cW + 2 * (nB - pB * args.cQ);
      b_voff[i] = nA < args.N ? (uint32_t)((krow * (int)args.ldb + sA) * ES) : OOB;
      b_voff2[i] = nB < args.N ? (uint32_t)((krow * (int)args.ldb + sB) * ES) : OOB;
      b_kch[i] = krow;
    } else {
      constexpr int CPRN = BN * ES / 16;
      const int krow = q / CPRN;
      int ch = q % CPRN;
      if constexpr (C::NC_DIRECT) ch ^= nc_swizzle(krow, C::VN) >> 4;      // slot q receives the chunk the swizzle maps there
      b_voff[i] = (uint32_t)((krow * (int)args.ldb + ch * EPC) * ES);
      b_kch[i] = krow;
    }
  }

  // ---- staging registers (global -> registers -> LDS)
  u32x4 ra[C::RSETS][C::DIRECT ? 1 : C::A_LOADS];
  u32x4 rb[C::RSETS][C::DIRECT ? 1 : C::B_LOADS * (C::BSRC == B_NCS2 ? 2 : 1)];

  // element-wise access of the convolution gather
  auto b_elem_bits = [&](int k, int col) -> uint32_t {
    if (col >= args.N || k >= Kx) return 0u;
    const int rs = args.cR * args.cS;
    const int c = k / rs, rr = (k - c * rs) / args.cS, ss = k - c * rs - rr * args.cS;
    const int pq = args.cP * args.cQ;
    const int img = col / pq, p = (col - img * pq) / args.cQ, q = col - img * pq - p * args.cQ;
    const int y = p * args.cStride - args.cPad + rr, x = q * args.cStride - args.cPad + ss;
    if (y < 0 || y >= args.cH || x < 0 || x >= args.cW) return 0u;
    const int64_t idx = (((int64_t)img * args.cC + c) * args.cH + y) * args.cW + x;
    if constexpr (ES == 4) return ((const uint32_t*)Bb)[idx];
    else return ((const uint16_t*)Bb)[idx];
  };
  // Operands that lie anywhere on element boundaries are fetched with the same 16-byte loads, at whatever address
  // a chunk starts (the memory path takes any).  `inner` says that no chunk of the tile holds an element beyond K and
  // none that is needed runs past the operand's last element: then that is all (rows and columns beyond the matrix
  // read other elements or zero and are never stored).  Otherwise, in the last one or two k tiles, a chunk is
  // fetched as the five aligned dwords around it -- the range check drops whole dwords, so the last element would
  // be lost to a dword that straddles the end -- shifted into place, and its elements beyond K are cleared (both
  // operands': a stray infinity times zero is not zero).
  // Element loads, two bytes a lane, were what bounded these instances: 2039 x 1511 x 1003 in bf16 took 100 us.
  auto load_chunks = [&](const __amdgpu_buffer_rsrc_t& r, uint32_t skew, const uint32_t* voff, u32x4* regs, auto chunks_tag) {
    constexpr int CHUNKS = decltype(chunks_tag)::value, LOADS = (CHUNKS + C::THREADS - 1) / C::THREADS;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      if (CHUNKS % C::THREADS != 0 && tid + i * C::THREADS >= CHUNKS) break;
      regs[i] = __builtin_amdgcn_raw_buffer_load_b128(r, voff[i] + skew, 0, 0);
    }
  };
  auto fetch_loose = [&](const char* first, int64_t bytes, bool inner, int k_left, const uint32_t* voff, const uint32_t* kch, u32x4* regs,
                         auto k_contiguous_tag, auto chunks_tag) {
    constexpr bool k_contiguous = decltype(k_contiguous_tag)::value;
    constexpr int CHUNKS = decltype(chunks_tag)::value, LOADS = (CHUNKS + C::THREADS - 1) / C::THREADS;
    if (k_left <= 0) return;                 // a k tile beyond the last: nothing of it is used
    uint32_t skew;
    const __amdgpu_buffer_rsrc_t r = loose_rsrc(first, bytes, skew);
    if (inner) {
      load_chunks(r, skew, voff, regs, chunks_tag);
    } else {
#pragma unroll
      for (int i = 0; i < LOADS; ++i) {
        if (CHUNKS % C::THREADS != 0 && tid + i * C::THREADS >= CHUNKS) break;
        const int left = k_left - (int)kch[i];             // k left from this chunk's first (or only) k
        const uint32_t off = left > 0 ? voff[i] + skew : OOB;
        u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off & ~3u, 0, 0);
        if constexpr (ES == 2) {
          const uint32_t w = __builtin_amdgcn_raw_buffer_load_b32(r, (off & ~3u) + 16u, 0, 0);
          const uint32_t half = off & 2u;
          const uint32_t d[5] = {v[0], v[1], v[2], v[3], w};
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_alignbyte(d[e + 1], d[e], half);
        }
        if constexpr (k_contiguous) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (ES == 4) v[e] = left > e ? v[e] : 0u;
            else v[e] &= left > 2 * e + 1 ? 0xffffffffu : (left > 2 * e ? 0xffffu : 0u);
          }
        }
        regs[i] = v;
      }
    }
  };
  auto pack_chunk = [&](auto&& elem) -> u32x4 {   // elem(e) for e in [0, EPC)
    u32x4 v;
    if constexpr (ES == 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = elem(e);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = elem(2 * e) | (elem(2 * e + 1) << 16);
    }
    return v;
  };

  // ---- fetch the k tile starting at k0: into registers, or straight into LDS stage `st`.
  // In a k-contiguous row a chunk beyond K would alias the next row, so those lanes are
  // sent out of range; this can only happen in the last k tile.
  auto fetch_a = [&](int k0, int st, int part = 0, int parts = 1, int set = 0) {
    const bool full = Kx - k0 >= BK;
    if constexpr (LOOSE_A) {
      if constexpr (C::ASRC == A_KC)
        fetch_loose(a_tile + (int64_t)k0 * ES, ((int64_t)(rows_valid - 1) * args.lda + (Kx - k0)) * ES, full, Kx - k0,
                    a_voff, a_kch, ra[set], std::true_type{}, std::integral_constant<int, C::A_CHUNKS>{});
      else
        fetch_loose(a_tile + (int64_t)k0 * args.lda * ES, ((int64_t)(Kx - k0 - 1) * args.lda + (args.M - m0)) * ES, Kx - k0 >= BK + EPC - 1, Kx - k0,
                    a_voff, a_kch, ra[set], std::false_type{}, std::integral_constant<int, C::A_CHUNKS>{});
    } else {
      const __amdgpu_buffer_rsrc_t r = rsrc_a(k0);
#pragma unroll
      for (int i = 0; i < C::A_LOADS; ++i) {
        if (C::A_CHUNKS % C::THREADS != 0 && tid + i * C::THREADS >= C::A_CHUNKS) break;
        if (i * parts < part * C::A_LOADS || i * parts >= (part + 1) * C::A_LOADS) continue;
        // (other direct staging is only launched for K a multiple of BK: every tile is full)
        const uint32_t off = (C::ASRC == A_MC || (C::DIRECT && !C::RING_16) || full || (int)a_kch[i] < Kx - k0) ? a_voff[i] : OOB;
        if constexpr (C::DIRECT)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (GENSOR_LDS void*)(lds + st * C::STAGE_BYTES + (i * C::THREADS + wave * 64) * 16),
                                                   16, off, 0, 0, 0);
        else
          ra[set][i] = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
      }
    }
  };
  auto fetch_b = [&](int k0, int st, int part = 0, int parts = 1, int set = 0) {
    const bool full = Kx - k0 >= BK;
    if constexpr (GATHER_B) {
#pragma unroll
      for (int i = 0; i < C::B_LOADS; ++i) {
        const int q = tid + i * C::THREADS;
        if (C::B_CHUNKS % C::THREADS != 0 && q >= C::B_CHUNKS) break;
        constexpr int CPRN = BN * ES / 16;
        const int krow = q / CPRN, ch = q % CPRN;
        rb[set][i] = pack_chunk([&](int e) { return b_elem_bits(k0 + krow, n0 + ch * EPC + e); });
      }
    } else if constexpr (LOOSE_B) {
      if constexpr (C::BSRC == B_KC)
        fetch_loose(b_tile + (int64_t)k0 * ES, ((int64_t)(cols_valid - 1) * args.ldb + (Kx - k0)) * ES, full, Kx - k0,
                    b_voff, b_kch, rb[set], std::true_type{}, std::integral_constant<int, C::B_CHUNKS>{});
      else
        fetch_loose(b_tile + (int64_t)k0 * args.ldb * ES, ((int64_t)(Kx - k0 - 1) * args.ldb + (args.N - n0)) * ES, Kx - k0 >= BK + EPC - 1, Kx - k0,
                    b_voff, b_kch, rb[set], std::false_type{}, std::integral_constant<int, C::B_CHUNKS>{});
    } else {
      const __amdgpu_buffer_rsrc_t r = rsrc_b(k0);
#pragma unroll
      for (int i = 0; i < C::B_LOADS; ++i) {
        if (C::B_CHUNKS % C::THREADS != 0 && tid + i * C::THREADS >= C::B_CHUNKS) break;
        if (i * parts < part * C::B_LOADS || i * parts >= (part + 1) * C::B_LOADS) continue;
        uint32_t off = b_voff[i];
        if constexpr (C::BSRC == B_KC && (!C::DIRECT || C::RING_16)) off = (full || (int)b_kch[i] < Kx - k0) ? off : OOB;
        if constexpr (C::DIRECT) {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (GENSOR_LDS void*)(lds + st * C::STAGE_BYTES + C::A_BYTES + (i * C::THREADS + wave * 64) * 16),
                                                   16, off, 0, 0, 0);
        } else if constexpr (C::BSRC == B_NCS2) {
          rb[set][2 * i] = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
          rb[set][2 * i + 1] = __builtin_amdgcn_raw_buffer_load_b128(r, b_voff2[i], 0, 0);
        } else {
          rb[set][i] = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        }
      }
    }
  };
  // Both operands of a k tile whose first k, and EPC - 1 more k rows than the tile has, lie inside K: no branch (fetch_loose's
  // `inner` of both).
  auto fetch_inner = [&](int k0, int set) {
    if constexpr (LOOSE_A && LOOSE_B) {
      uint32_t skew;
      const __amdgpu_buffer_rsrc_t r = C::ASRC == A_KC ? loose_rsrc(a_tile + (int64_t)k0 * ES, ((int64_t)(rows_valid - 1) * args.lda + (Kx - k0)) * ES, skew)
          : loose_rsrc(a_tile + (int64_t)k0 * args.lda * ES, ((int64_t)(Kx - k0 - 1) * args.lda + (args.M - m0)) * ES, skew);
      load_chunks(r, skew, a_voff, ra[set], std::integral_constant<int, C::A_CHUNKS>{});
      const __amdgpu_buffer_rsrc_t q = C::BSRC == B_KC ? loose_rsrc(b_tile + (int64_t)k0 * ES, ((int64_t)(cols_valid - 1) * args.ldb + (Kx - k0)) * ES, skew)
          : loose_rsrc(b_tile + (int64_t)k0 * args.ldb * ES, ((int64_t)(Kx - k0 - 1) * args.ldb + (args.N - n0)) * ES, skew);
      load_chunks(q, skew, b_voff, rb[set], std::integral_constant<int, C::B_CHUNKS>{});
    }
  };
  // ---- registers -> LDS stage `st`
  auto commit = [&](int st, int set = 0) {
    if constexpr (!C::DIRECT) {
      GENSOR_LDS char* abase = lds + st * C::STAGE_BYTES;
      GENSOR_LDS char* bbase = abase + C::A_BYTES;
#pragma unroll
      for (int i = 0; i < C::A_LOADS; ++i) {
        const int q = tid + i * C::THREADS;
        if (C::A_CHUNKS % C::THREADS != 0 && q >= C::A_CHUNKS) break;
        if constexpr (C::ASRC == A_KC) {
          *(GENSOR_LDS u32x4*)(abase + q * 16) = ra[set][i];
        } else {
          constexpr int CPRM = BM * ES / 16;
          *(GENSOR_LDS u32x4*)(abase + (q / CPRM) * C::PITCH_M + (q % CPRM) * 16) = ra[set][i];
        }
      }
#pragma unroll
      for (int i = 0; i < C::B_LOADS; ++i) {
        const int q = tid + i * C::THREADS;
        if (C::B_CHUNKS % C::THREADS != 0 && q >= C::B_CHUNKS) break;
        if constexpr (C::BSRC == B_KC) {
          *(GENSOR_LDS u32x4*)(bbase + q * 16) = rb[set][i];
        } else if constexpr (C::BSRC == B_NCS2) {
          // keep every other element of the two 16-byte runs
          constexpr int CPRN = BN * ES / 16;
          const u32x4 v0 = rb[set][2 * i], v1 = rb[set][2 * i + 1];
          u32x4 o;
          if constexpr (ES == 4) {
            o[0] = v0[0]; o[1] = v0[2]; o[2] = v1[0]; o[3] = v1[2];
          } else {
            o[0] = __builtin_amdgcn_perm(v0[1], v0[0], 0x05040100u);
            o[1] = __builtin_amdgcn_perm(v0[3], v0[2], 0x05040100u);
            o[2] = __builtin_amdgcn_perm(v1[1], v1[0], 0x05040100u);
            o[3] = __builtin_amdgcn_perm(v1[3], v1[2], 0x05040100u);
          }
          *(GENSOR_LDS u32x4*)(bbase + (q / CPRN) * C::PITCH_N + (q % CPRN) * 16) = o;
        } else {
          constexpr int CPRN = BN * ES / 16;
          *(GENSOR_LDS u32x4*)(bbase + (q / CPRN) * C::PITCH_N + (q % CPRN) * 16) = rb[set][i];
        }
      }
    }
  };
  // all of this wave's direct deposits have landed (vmcnt(0); expcnt and lgkmcnt untouched)
  auto wait_deposits = [&]() {
    if constexpr (C::DIRECT) __builtin_amdgcn_s_waitcnt(0x0F70);
  };

  // ---- fragments.  fa[b] / fb[b] are two register sets so that the reads of k step s+1
  // are in flight while the MFMAs of step s issue.
  const int frow = lane % MB;          // row / column inside an MFMA block
  const int fgrp = lane / MB;          // which chunk of the k group this lane holds
  auto block_row = [&](int bi) { return wave_m * C::WM + bi * MB; };   // first row of MFMA block bi of this wave inside the BM tile
  auto block_col = [&](int bj) { return wave_n * C::WN + bj * MB; };
  // One wave per SIMD (four waves of 128x128): nothing else covers a stall, so fragments are read
  // two k steps ahead (one register set per k step of a tile) and the barrier sits in front of step 2
  // (4096^3 on all-zero operands, where the power limit does not interfere: 88.0 -> 81.4 us; 8192^3 on
  // the benchmark's operands: 971 -> 910 us, against 950 us for eight waves of 128x64).
  constexpr bool DEEP = C::DIRECT && C::STAGES == 2 && C::KSTEPS == 4 && C::MBLK * C::NBLK >= 16;
  constexpr int FSETS = DEEP ? 4 : 2;
  u32x4 fa[FSETS][C::MBLK], fb[FSETS][C::NBLK];
  // Direct staging with an n-contiguous 16-bit B: the transposing fragment reads are issued from inline assembly.
  // A compiler-issued LDS read that it cannot tell apart from the destinations of the direct loads in flight is
  // preceded by a wait for ALL of them (vmcnt(0)), which it does for the transposing-read builtin: every k tile
  // then waited out the full latency of the loads just issued for the next one.  The assembly reads are invisible
  // to the compiler's counter bookkeeping, so the kernel waits for them itself: `settle` below, in front of the
  // MFMAs that consume a register set.  LDS operations complete in issue order and the statements are volatile,
  // hence ordered: "at most N outstanding", with N no more than the number of such reads issued after the awaited
  // ones, means the awaited ones have landed.  The halves stay separate values until that wait (a copy of a pending
  // register would read stale data); the compiler's own waits only get more conservative by operations it does not see.
  // An m-contiguous A staged directly is read the same way, and a k-contiguous one beside such a B too: left to the
  // compiler, its waits counted only its own reads and so waited for reads issued a moment earlier, in every k step
  // (8192 x 768 x 3072 f16, 128x256 ring: 46.5 -> 42.7 us, eight-wave 128x128 tile 49.8 -> 46.9).
  constexpr bool ASM_A = C::MC_DIRECT, ASM_B = C::NC_DIRECT && ES == 2, ASM_TR = ASM_A || ASM_B;
  u32x2 fal[ASM_A ? FSETS : 1][ASM_A ? C::MBLK : 1], fah[ASM_A ? FSETS : 1][ASM_A ? C::MBLK : 1];
  u32x2 fbl[ASM_B ? FSETS : 1][ASM_B ? C::NBLK : 1], fbh[ASM_B ? FSETS : 1][ASM_B ? C::NBLK : 1];
  // The two transposing reads of one block from an unpadded, XOR-swizzled tile stored [k][rows].  The swizzle of a lane's
  // k rows is the same in every k step and four rows further down, so those are immediate offsets.
  auto issue_transposed = [&](GENSOR_LDS char* base, auto pitch_tag, int first, auto ks_tag, int v, u32x2& lo, u32x2& hi) {
    constexpr int pitch = decltype(pitch_tag)::value, ks = decltype(ks_tag)::value;
    const int g = lane >> 4, s = lane & 15;
    const int krow = (MB == 32 ? (g >> 1) * 8 : g * 8) + (s >> 2);
    const int col = first + (MB == 32 ? (g & 1) * 16 : 0) + (s & 3) * 4;
    const uint32_t at = (uint32_t)(uintptr_t)(base + krow * pitch + ((col * 2) ^ nc_swizzle(krow, v)));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(at), "n"(ks * C::KG * pitch));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(at), "n"((ks * C::KG + 4) * pitch));
  };
  // Fragment of one MFMA block from a tile stored [k][rows] (an n-contiguous B or an m-contiguous A), `first` =
  // the block's first row/column inside the tile, `direct` = the tile is unpadded and XOR-swizzled.
  auto read_transposed = [&](GENSOR_LDS char* base, int pitch, int first, int ks, auto direct_tag, int v) -> u32x4 {
    constexpr bool direct = decltype(direct_tag)::value;
    if constexpr (ES == 4) {
      // fp32: element t of this lane's chunk is k = ks*KG + fgrp*4 + t
      const int col = first + frow;
      u32x4 r;
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        const int kr = ks * C::KG + fgrp * 4 + tt;
        const int cb = direct ? ((col * 4) ^ nc_swizzle(kr, v)) : col * 4;
        r[tt] = *(GENSOR_LDS uint32_t*)(base + kr * pitch + cb);
      }
      return r;
    } else {
      // 16-bit: two transposing reads.  In each 16-lane group, lane s fetches 4 consecutive rows/columns of
      // k row (s/4) and receives, for row/column s, the 4 consecutive k of the group's k rows.
      const int g = lane >> 4, s = lane & 15;
      int krow, col;
      if constexpr (MB == 32) {    // groups: (g%2) picks the 16-wide half, (g/2) the 8-deep k half
        krow = ks * C::KG + (g >> 1) * 8 + (s >> 2);
        col = first + (g & 1) * 16 + (s & 3) * 4;
      } else {                     // 16x16 blocks: group g holds k = 8g..8g+7
        krow = ks * C::KG + g * 8 + (s >> 2);
        col = first + (s & 3) * 4;
      }
      const int cb0 = direct ? ((col * 2) ^ nc_swizzle(krow, v)) : col * 2;
      const int cb1 = direct ? ((col * 2) ^ nc_swizzle(krow + 4, v)) : col * 2;
      GENSOR_LDS char* p = base + krow * pitch;
      s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GENSOR_LDS s16x4*)(p + cb0));
      s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GENSOR_LDS s16x4*)(p + 4 * pitch + cb1));
      u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
      u32x4 r = {l2[0], l2[1], h2[0], h2[1]};
      return r;
    }
  };
  auto read_frags_asm = [&](int st, auto ks_tag, int buf) {
    constexpr int ks = decltype(ks_tag)::value;
    GENSOR_LDS char* abase = lds + st * C::STAGE_BYTES;
    GENSOR_LDS char* bbase = abase + C::A_BYTES;
    const int ch = ks * C::LANE_GROUPS + fgrp;
    static_for<C::MBLK>([&](auto bi) {
      if constexpr (ASM_A) {
        issue_transposed(abase, std::integral_constant<int, C::PITCH_M>{}, block_row(bi), ks_tag, C::VM, fal[buf][bi], fah[buf][bi]);
      } else {
        // rows MB apart share their swizzle: blocks are immediate offsets
        const int row = block_row(0) + frow;
        const uint32_t at = (uint32_t)(uintptr_t)(abase + row * C::PITCH_K + swizzled_chunk(row, ch, C::RPP, C::VM) * 16);
        u32x4& frag = fa[buf][bi];
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(frag) : "v"(at), "n"(decltype(bi)::value * MB * C::PITCH_K));
      }
    });
    static_for<C::NBLK>([&](auto bj) {
      if constexpr (ASM_B) {
        issue_transposed(bbase, std::integral_constant<int, C::PITCH_N>{}, block_col(bj), ks_tag, C::VN, fbl[buf][bj], fbh[buf][bj]);
      } else {
        const int row = block_col(0) + frow;
        const uint32_t at = (uint32_t)(uintptr_t)(bbase + row * C::PITCH_K + swizzled_chunk(row, ch, C::RPP, C::VN) * 16);
        u32x4& frag = fb[buf][bj];
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(frag) : "v"(at), "n"(decltype(bj)::value * MB * C::PITCH_K));
      }
    });
  };
  auto read_frags = [&](int st, int ks, int buf) {
    if constexpr (ASM_TR) {
      // (ks is a constant at every call once the k steps are unrolled: one of these remains)
      static_for<C::KSTEPS>([&](auto k) { if (ks == decltype(k)::value) read_frags_asm(st, k, buf); });
      return;
    }
    GENSOR_LDS char* abase = lds + st * C::STAGE_BYTES;
    GENSOR_LDS char* bbase = abase + C::A_BYTES;
    const int ch = ks * C::LANE_GROUPS + fgrp;
#pragma unroll
    for (int bi = 0; bi < C::MBLK; ++bi) {
      if constexpr (C::ASRC == A_KC) {
        const int row = block_row(bi) + frow;
        fa[buf][bi] = *(GENSOR_LDS u32x4*)(abase + row * C::PITCH_K + swizzled_chunk(row, ch, C::RPP, C::VM) * 16);
      } else {
        fa[buf][bi] = read_transposed(abase, C::PITCH_M, block_row(bi), ks, std::false_type{}, C::VM);
      }
    }
#pragma unroll
    for (int bj = 0; bj < C::NBLK; ++bj) {
      if constexpr (C::BSRC == B_KC) {
        const int row = block_col(bj) + frow;
        fb[buf][bj] = *(GENSOR_LDS u32x4*)(bbase + row * C::PITCH_K + swizzled_chunk(row, ch, C::RPP, C::VN) * 16);
      } else {
        fb[buf][bj] = read_transposed(bbase, C::PITCH_N, block_col(bj), ks, std::integral_constant<bool, C::NC_DIRECT>{}, C::VN);
      }
    }
  };
  // groups: how many later read_frags calls (READS LDS reads each) have been issued since the one that filled register
  // set buf -- a lower bound; 0 waits for every LDS operation
  auto settle = [&](int buf, auto groups_tag) {
    if constexpr (ASM_TR) {
      constexpr int READS = (ASM_A ? 2 : 1) * C::MBLK + (ASM_B ? 2 : 1) * C::NBLK;
      constexpr int N = decltype(groups_tag)::value * READS > 15 ? 15 : decltype(groups_tag)::value * READS;
      bool waited = false;
      auto take = [&](auto& x) {
        if (!waited) asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N));
        else asm volatile("" : "+v"(x));
        waited = true;
      };
#pragma unroll
      for (int bi = 0; bi < C::MBLK; ++bi) {
        if constexpr (ASM_A) {
          take(fal[buf][bi]);
          take(fah[buf][bi]);
          const u32x4 v = {fal[buf][bi][0], fal[buf][bi][1], fah[buf][bi][0], fah[buf][bi][1]};
          fa[buf][bi] = v;
        } else {
          take(fa[buf][bi]);
        }
      }
#pragma unroll
      for (int bj = 0; bj < C::NBLK; ++bj) {
        if constexpr (ASM_B) {
          take(fbl[buf][bj]);
          take(fbh[buf][bj]);
          const u32x4 v = {fbl[buf][bj][0], fbl[buf][bj][1], fbh[buf][bj][0], fbh[buf][bj][1]};
          fb[buf][bj] = v;
        } else {
          take(fb[buf][bj]);
        }
      }
    }
  };
  // Workgroup barrier of the k loop.  The transposing reads issued from assembly must have left the LDS before
  // another wave may overwrite the stage they read; the compiler does not know of them, so the wait is explicit.
  auto block_sync = [&]() {
    if constexpr (ASM_TR) __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0); the other counters untouched
    __syncthreads();
  };
  // (`at`: the k step, counted over the k tiles of the register sets, where a block has several chains)
  auto mma = [&](int buf, auto groups_tag, int at = 0) {
    settle(buf, groups_tag);
#pragma unroll
    for (int bi = 0; bi < C::MBLK; ++bi)
#pragma unroll
      for (int bj = 0; bj < C::NBLK; ++bj) {
        if constexpr (CHAINS > 1 && ES == 4 && MB == 16) {
#pragma unroll
          for (int t = 0; t < 4; ++t) MF::step(fa[buf][bi], fb[buf][bj], t, chain((4 * at + t) % CHAINS, bi, bj));
        } else {
          MF::run(fa[buf][bi], fb[buf][bj], chain(at % CHAINS, bi, bj));
        }
      }
  };

  // Scheduling hint for one k step: issue the fragment reads of the next step in small
  // groups in front of each MFMA of this step, so that they complete under matrix work.
  auto interleave = [&]() {
    constexpr int NM = C::MBLK * C::NBLK * (ES == 4 ? 4 : 1);
    constexpr int NR = C::MBLK * (C::ASRC == A_KC ? 1 : (ES == 4 ? 4 : 2)) + C::NBLK * (C::BSRC == B_KC ? 1 : (ES == 4 ? 4 : 2));
    constexpr int RPM = (NR + NM - 1) / NM;
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);   // LDS reads
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // one MFMA
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // the same with the global loads of this step between the MFMAs as well.  One wave per SIMD
  // (`separate`): the fragment reads in front of the first MFMAs, then one load per MFMA, so that
  // no gap between two MFMAs has to issue both a read and a load.  Two waves per SIMD measure better
  // with a load and a read per gap, loads first.
  auto interleave_vmem = [&](auto separate_tag) {
    constexpr bool separate = decltype(separate_tag)::value;
    constexpr int NM = C::MBLK * C::NBLK * (ES == 4 ? 4 : 1);
    constexpr int NR = C::MBLK * (C::ASRC == A_KC ? 1 : (ES == 4 ? 4 : 2)) + C::NBLK * (C::BSRC == B_KC ? 1 : (ES == 4 ? 4 : 2));
    constexpr int RPM = (NR + NM - 1) / NM;
    constexpr int READ_SLOTS = (NR + RPM - 1) / RPM;
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      if constexpr (separate) {
        if (i < READ_SLOTS) __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);   // LDS reads
        else __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                     // one global load
      } else {
        __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            // one MFMA
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- main loop over k tiles.  Tile kt+1 is fetched while tile kt is multiplied; its
  // first fragments are read right after the barrier, under the MFMAs of the last k step
  // of tile kt, so that the barrier and the LDS latency are covered by matrix work.
  const int nk = (Kx + BK - 1) / BK;
  constexpr bool PIPE = (C::KSTEPS % 2 == 0) && C::STAGES == 2;
  if constexpr (C::STAGES <= 2 && !C::ALTERNATE) {
    fetch_a(0, 0);
    fetch_b(0, 0);
    if constexpr (C::RSETS == 2) {
      fetch_a(BK, 0, 0, 1, 1);
      fetch_b(BK, 0, 0, 1, 1);
    }
    commit(0);
    wait_deposits();
    __syncthreads();
  }
  if constexpr (C::ALTERNATE) {
    // Large tiles run into the chip's power limit, which 16x16x32 products reach at 1957 TFLOP/s and 32x32x16 ones at 1705
    // (registers only, uniform operands), but only from two waves per SIMD (one: 1784).  So: eight waves of 16x16 blocks, and so
    // that the two waves of a SIMD do not wait for the LDS together, the four waves of the upper half of the tile (group
    // 0) and the four of the lower half (group 1) alternate.  Time is cut into slots by barriers.  In slot 2t group 0
    // multiplies k tile t, all of whose fragments it holds, while group 1 reads its fragments of tile t; in slot 2t+1 group
    // 1 multiplies and group 0 reads tile t+1.  A multiplying wave issues nothing but MFMAs, in an order in which each one
    // shares an operand with the one before (2 % more under the power limit).  The direct loads go out between the
    // fragment reads, 32 a slot; a slot of 48 followed by one of 16 took 1220 cycles instead of 1080, loads behind the reads 1440.
    //   A(t), in stage t % 2: group g reads only its own half.  In slot 2t group 1 requests the upper half of A(t+2) (group 0 read
    //   that of A(t) in slot 2t-1), in slot 2t+1 group 0 the lower half (group 1 read it in slot 2t).
    //   B(t), in stage t % 3: both read it, the later in slot 2t.  Group 1 requests half of B(t+2) in slot 2t, group 0 the other half
    //   of B(t+3) in slot 2t+1.
    // Every request has at least two slots before the barrier behind which it is read.  Each wave waits for its own
    // requests in front of that barrier; they land in issue order, so the waits are counts.
    // 4096^3 f16 118 -> 104 us (all-zero operands 79 -> 70), 8192^3 911 -> 800 (771 -> 575), against four 128x128 waves of 32x32 blocks.
    // Raising the wave priority while multiplying starves the readers (108 us on zeros); MFMAs behind the barrier of their
    // slot, to cover it, delay the next slot's reads (81 us).
    // Tiles of 192 columns (NarrowCfg): a group's four waves are two by two of 64x96 instead of four of 128x64 side by side, which
    // reads 160 rows a wave and k tile where 128x48 waves would read 176.
    static_assert(C::KSTEPS == 2 && C::A_BYTES == 32768 && C::B_BYTES == BN * 128, "two k steps; 32 KiB of A, 128 bytes of B a column");
    constexpr int WM2 = C::WAVES_M / 2;                        // rows of waves in a group
    constexpr int NA = 4, NBR = BN / 64;                       // a wave's requests of each operand: 1 KiB runs of one half of its tile
    constexpr int NB = C::MBLK * C::NBLK;
    const int group = wave >> 2, w4 = wave & 3;
    auto stage_a = [&](int t) { return lds + (t & 1) * C::A_BYTES; };
    auto stage_b = [&](int t3) { return lds + 2 * C::A_BYTES + t3 * C::B_BYTES; };
    // This wave's requests: 1 KiB runs of one half of each operand's tile.  (Chunks 512 apart have the same swizzle, but for the
    // rows of 24 chunks of an n-contiguous B.)
    // Rows of an n-contiguous B are whole 128-byte groups; of four k rows read together the pitch of an odd number of groups
    // already spreads two over the banks, and only the other bit is left to the swizzle, which stays inside a group.
    auto swizzle_b = [&](int krow) -> int {
      if constexpr (BN * ES % 256 == 0) return nc_swizzle(krow, C::VN);
      else return C::VN >= 4 ? ((krow >> 1 & 1) << 6) ^ ((krow >> 3 & 1) << 5) : 0;
    };
    // An m-contiguous A is kept as two halves [k][128 rows]: a run has to be contiguous in the LDS and in one half.
    const int half_a = 1 - group, half_b = group;
    constexpr bool ROWS_24 = C::BSRC != B_KC && NBR == 3;
    constexpr int VB = ROWS_24 ? 3 : 2;
    uint32_t va[2], vb[VB], step_a, step_b = 0;
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      const int q = (i * 4 + w4) * 64 + lane;                  // chunk inside the half
      if (i >= 2) {
      } else if constexpr (C::ASRC == A_KC) {
        const int row = half_a * 128 + q / C::CPR;
        va[i] = (uint32_t)((row * (int)args.lda + swizzled_chunk(row, q % C::CPR, C::RPP, C::VM) * EPC) * ES);
        step_a = (uint32_t)((512 / C::CPR) * (int)args.lda * ES);
      } else {
        const int krow = q / 16, ch = (q % 16) ^ (nc_swizzle(krow, C::VM) >> 4);
        va[i] = (uint32_t)((krow * (int)args.lda + half_a * 128 + ch * EPC) * ES);
        step_a = (uint32_t)((512 / 16) * (int)args.lda * ES);
      }
      const int q2 = half_b * (NBR * 256) + q;
      if constexpr (C::BSRC == B_KC) {
        const int row = q2 / C::CPR;
        vb[i] = (uint32_t)((row * (int)args.ldb + swizzled_chunk(row, q2 % C::CPR, C::RPP, C::VN) * EPC) * ES);
        step_b = (uint32_t)((512 / C::CPR) * (int)args.ldb * ES);
      } else {
        constexpr int CPRN = BN * ES / 16;
        const int krow = q2 / CPRN, ch = (q2 % CPRN) ^ (swizzle_b(krow) >> 4);
        vb[i] = (uint32_t)((krow * (int)args.ldb + ch * EPC) * ES);
        if constexpr (!ROWS_24) step_b = (uint32_t)((512 / CPRN) * (int)args.ldb * ES);
      }
    }
    // K need not be a multiple of BK: k rows beyond it lie beyond the descriptor; a chunk of a k-contiguous row that does
    // would alias the next row and is sent out of range (an offset at OOB stays there when a step is added).
    const int k_a = (int)((lane & 7) ^ (((w4 * 8 + (lane >> 3)) / C::RPP) % C::VM)) * EPC;
    const int k_b = (int)((lane & 7) ^ (((w4 * 8 + (lane >> 3)) / C::RPP) % C::VN)) * EPC;
    struct Offsets { uint32_t at[3]; };
    auto offsets_a = [&](int t) {
      if constexpr (C::ASRC != A_KC) return Offsets{{va[0], va[1], 0}};
      const bool in = k_a < Kx - t * BK;
      return Offsets{{in ? va[0] : OOB, in ? va[1] : OOB, 0}};
    };
    auto offsets_b = [&](int t) {
      if constexpr (C::BSRC != B_KC) return Offsets{{vb[0], vb[1], vb[VB - 1]}};
      const bool in = k_b < Kx - t * BK;
      return Offsets{{in ? vb[0] : OOB, in ? vb[1] : OOB, 0}};
    };
    auto load_a = [&](const __amdgpu_buffer_rsrc_t& r, const Offsets& o, GENSOR_LDS char* stage, int i) {
      load_to_lds(r, stage + (half_a * 16 + i * 4 + w4) * 1024, o.at[i & 1] + (uint32_t)(i >> 1) * step_a);
    };
    auto load_b = [&](const __amdgpu_buffer_rsrc_t& r, const Offsets& o, GENSOR_LDS char* stage, int i) {
      load_to_lds(r, stage + (half_b * (NBR * 4) + i * 4 + w4) * 1024, ROWS_24 ? o.at[i] : o.at[i & 1] + (uint32_t)(i >> 1) * step_b);
    };
    auto request_a = [&](int t) {
      const __amdgpu_buffer_rsrc_t r = rsrc_a(t * BK);
      const Offsets o = offsets_a(t);
#pragma unroll
      for (int i = 0; i < NA; ++i) load_a(r, o, stage_a(t), i);
    };
    auto request_b = [&](int t, int t3) {
      const __amdgpu_buffer_rsrc_t r = rsrc_b(t * BK);
      const Offsets o = offsets_b(t);
#pragma unroll
      for (int i = 0; i < NBR; ++i) load_b(r, o, stage_b(t3), i);
    };
    auto pin = [&]() { __builtin_amdgcn_sched_barrier(0); };
    auto end_slot = [&]() { pin(); __builtin_amdgcn_s_barrier(); pin(); };
    // at most n of this wave's requests outstanding
    auto landed = [&](auto n_tag) {
      constexpr int n = decltype(n_tag)::value;
      pin();
      __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
    };
    // Where this lane reads inside a stage.  A tile's rows are 128 (k-contiguous), 256 (m-contiguous: half a tile), 384 or 512
    // bytes and blocks and k steps differ in bits that the swizzle only XORs, so every read's address is one exclusive or
    // away from the lane's first and one immediate offset.
    auto lane_k = [&](int row, int v) { return (uint32_t)(row * C::PITCH_K + swizzled_chunk(row, fgrp, C::RPP, v) * 16); };
    const int tr_row = (lane >> 4) * 8 + ((lane & 15) >> 2);
    auto lane_tr = [&](int pitch, int first_byte, int swizzle) { return (uint32_t)(tr_row * pitch + ((first_byte + (lane & 3) * 8) ^ swizzle)); };
    uint32_t lane_a = ASM_A ? group * (C::A_BYTES / 2) + lane_tr(256, wave_m % WM2 * C::WM * ES, nc_swizzle(tr_row, C::VM))
                            : lane_k(block_row(0) + frow, C::VM);
    // (a wave's 96 columns start on half a 128-byte group: one address for each two blocks)
    constexpr int LB = ASM_B && C::WN % 64 != 0 ? C::NBLK / 2 : 1;
    uint32_t lane_b[LB];
#pragma unroll
    for (int p = 0; p < LB; ++p)
      lane_b[p] = ASM_B ? lane_tr(BN * ES, block_col(2 * p) * ES, swizzle_b(tr_row)) : lane_k(block_col(0) + frow, C::VN);
    auto read_tr = [&](uint32_t at, auto pitch_tag, auto ks_tag, u32x2& lo, u32x2& hi) {
      constexpr int pitch = decltype(pitch_tag)::value, k = decltype(ks_tag)::value * C::KG;
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(at), "n"(k * pitch));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(at), "n"((k + 4) * pitch));
    };
    auto read_k = [&](GENSOR_LDS char* at, auto off_tag, u32x4& frag) {
      constexpr int off = decltype(off_tag)::value;
      if constexpr (ASM_TR) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(frag) : "v"((uint32_t)(uintptr_t)at), "n"(off));
      else frag = *(GENSOR_LDS u32x4*)(at + off);
    };
    // fragments of one block of one k step
    auto read_a = [&](GENSOR_LDS char* stage, auto ks_tag, auto bi_tag) {
      constexpr int ks = decltype(ks_tag)::value, bi = decltype(bi_tag)::value;
      if constexpr (ASM_A) read_tr((uint32_t)(uintptr_t)(stage + (lane_a ^ (bi * MB * ES))), std::integral_constant<int, 256>{}, ks_tag, fal[ks][bi], fah[ks][bi]);
      else read_k(stage + (lane_a ^ (ks * 64)), std::integral_constant<int, bi * MB * C::PITCH_K>{}, fa[ks][bi]);
    };
    auto read_b = [&](GENSOR_LDS char* stage, auto ks_tag, auto bj_tag) {
      constexpr int ks = decltype(ks_tag)::value, bj = decltype(bj_tag)::value;
      if constexpr (ASM_B) read_tr((uint32_t)(uintptr_t)(stage + (lane_b[LB > 1 ? bj / 2 : 0] ^ ((LB > 1 ? bj % 2 : bj) * MB * ES))), std::integral_constant<int, BN * ES>{}, ks_tag, fbl[ks][bj], fbh[ks][bj]);
      else read_k(stage + (lane_b[0] ^ (ks * 64)), std::integral_constant<int, bj * MB * C::PITCH_K>{}, fb[ks][bj]);
    };
    // A reading slot: the fragments of a tile, with this wave's requests of each operand between them (`ra`, `rb`: the tiles
    // requested), then the wait for all but the youngest `left` requests and the barrier.
    auto read_slot = [&](int t, int t3, auto ra_tag, int ra, auto rb_tag, int rb, int rb3, auto left_tag) {
      constexpr bool want_a = decltype(ra_tag)::value, want_b = decltype(rb_tag)::value;
      const __amdgpu_buffer_rsrc_t qa = rsrc_a(want_a ? ra * BK : 0), qb = rsrc_b(want_b ? rb * BK : 0);
      const Offsets oa = offsets_a(ra), ob = offsets_b(rb);
      GENSOR_LDS char* ta = stage_a(t);
      GENSOR_LDS char* tb = stage_b(t3);
      asm volatile("" : "+v"(lane_a), "+v"(lane_b[0]));        // (kept from computing all addresses once: they do not fit the registers)
      constexpr int ITEMS = C::MBLK + C::NBLK;
      static_for<2 * ITEMS>([&](auto j_tag) {
        constexpr int j = decltype(j_tag)::value, e = j % ITEMS;
        constexpr std::integral_constant<int, j / ITEMS> ks{};
        if constexpr (e < C::NBLK) read_b(tb, ks, std::integral_constant<int, e>{});
        else read_a(ta, ks, std::integral_constant<int, e - C::NBLK>{});
        constexpr int l = (j + 1) * (NA + NBR) / (2 * ITEMS) - 1;          // the request behind this read
        if constexpr ((j + 1) * (NA + NBR) / (2 * ITEMS) > j * (NA + NBR) / (2 * ITEMS)) {
          pin();
          if constexpr (l < NA && want_a) load_a(qa, oa, stage_a(ra), l);
          if constexpr (l >= NA && want_b) load_b(qb, ob, stage_b(rb3), l - NA);
          pin();
        }
      });
      landed(left_tag);
      __builtin_amdgcn_s_waitcnt(0xC07F);                      // the fragments are here: their stage may be overwritten
      end_slot();
    };
    auto multiply = [&]() {
      settle(0, std::integral_constant<int, 0>{});
      settle(1, std::integral_constant<int, 0>{});
#pragma unroll
      for (int x = 0; x < 2 * NB; ++x) {
        const int ks = x / NB, bi = x % NB / C::NBLK, j = x % C::NBLK, bj = (bi & 1) ? C::NBLK - 1 - j : j;
        MF::run(fa[ks][bi], fb[ks][bj], acc[bi][bj]);
      }
      pin();
    };
    auto third = [&](int t3, int by) { return t3 + by >= 3 ? t3 + by - 3 : t3 + by; };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr std::integral_constant<int, 0> all{};
    constexpr std::integral_constant<int, NA> but_a{};         // all but the requests of one tile of A, of B, of both, and of another B
    constexpr std::integral_constant<int, NBR> but_b{};
    constexpr std::integral_constant<int, NA + NBR> but_ab{};
    constexpr std::integral_constant<int, NA + 2 * NBR> but_ab2{};
    int t = 0, t3 = 0;                                         // k tile, and t % 3
    request_a(0);
    request_b(0, 0);
    if (group == 0) {
      if (nk > 1) {
        request_b(1, 1);
        landed(but_b);
      } else {
        landed(all);
      }
      end_slot();
      if (nk > 2) read_slot(0, 0, yes, 1, yes, 2, 2, but_ab2);
      else if (nk > 1) read_slot(0, 0, yes, 1, no, 0, 0, but_a);
      else read_slot(0, 0, no, 0, no, 0, 0, all);
      for (; t + 3 < nk; ++t, t3 = third(t3, 1)) {
        multiply();
        landed(but_ab);
        end_slot();
        read_slot(t + 1, third(t3, 1), yes, t + 2, yes, t + 3, t3, but_ab2);
      }
      if (t + 2 < nk) {
        multiply();
        landed(but_ab);
        end_slot();
        read_slot(t + 1, third(t3, 1), yes, t + 2, no, 0, 0, but_ab);
        ++t;
        t3 = third(t3, 1);
      }
      if (t + 1 < nk) {
        multiply();
        landed(all);
        end_slot();
        read_slot(t + 1, third(t3, 1), no, 0, no, 0, 0, all);
      }
      multiply();
      end_slot();
      end_slot();
    } else {
      if (nk > 1) {
        request_a(1);
        request_b(1, 1);
        landed(but_ab);
      } else {
        landed(all);
      }
      end_slot();
      end_slot();
      for (; t + 2 < nk; ++t, t3 = third(t3, 1)) {
        read_slot(t, t3, yes, t + 2, yes, t + 2, third(t3, 2), but_ab);
        multiply();
        end_slot();
      }
      for (; t < nk; ++t, t3 = third(t3, 1)) {
        read_slot(t, t3, no, 0, no, 0, 0, all);
        multiply();
        end_slot();
      }
    }
  } else if constexpr (DEEP) {
    // By the barrier in front of step 2 every wave has read (and received) steps 2 and 3 of this
    // tile, so its stage is free: the loads of tile kt+2 go out right behind the barrier, over
    // steps 2 and 3 and between their MFMAs, a whole k tile before they are needed.
    auto k_tile = [&](int kt, auto next_tag, auto fetch_tag) {
      constexpr bool has_next = decltype(next_tag)::value, has_fetch = decltype(fetch_tag)::value;
      const int cur = kt & 1, nxt = cur ^ 1;
      read_frags(cur, 2, 2);
      mma(0, std::integral_constant<int, 2>{});
      interleave();
      read_frags(cur, 3, 3);
      mma(1, std::integral_constant<int, 2>{});
      interleave();
      if constexpr (has_next) {
        wait_deposits();
        block_sync();
        read_frags(nxt, 0, 0);
        if constexpr (has_fetch) {
          fetch_a((kt + 2) * BK, cur, 0, 2);
          fetch_b((kt + 2) * BK, cur, 0, 2);
        }
      }
      mma(2, std::integral_constant<int, has_next ? 2 : 1>{});
      if constexpr (has_fetch) interleave_vmem(std::true_type{});
      else interleave();
      if constexpr (has_next) {
        read_frags(nxt, 1, 1);
        if constexpr (has_fetch) {
          fetch_a((kt + 2) * BK, cur, 1, 2);
          fetch_b((kt + 2) * BK, cur, 1, 2);
        }
      }
      mma(3, std::integral_constant<int, has_next ? 2 : 0>{});
      if constexpr (has_fetch) interleave_vmem(std::true_type{});
      else interleave();
    };
    if (nk > 1) {
      fetch_a(BK, 1);
      fetch_b(BK, 1);
    }
    read_frags(0, 0, 0);
    read_frags(0, 1, 1);
    for (int kt = 0; kt + 2 < nk; ++kt) k_tile(kt, std::true_type{}, std::true_type{});
    if (nk > 1) k_tile(nk - 2, std::true_type{}, std::false_type{});
    k_tile(nk - 1, std::false_type{}, std::false_type{});
  } else if constexpr (C::STAGES > 2) {
    // Ring of STAGES buffers: STAGES-1 k tiles are in flight, so a tile has STAGES-1 tile times to
    // arrive.  Loads complete in issue order, hence "tile kt+1 has landed" is "at most the loads
    // of the STAGES-2 younger tiles are outstanding"; near the end of k fewer tiles are in flight
    // and the wait is for all of them.  Three copies of the body (steady state, draining, last
    // tile) keep those facts compile-time.  The stage refilled at the top of tile kt is the one
    // read during tile kt-1, which every wave left before the barrier that ended that tile.
    constexpr int S = C::STAGES;
    constexpr int LPT = C::A_LOADS + C::B_LOADS;             // loads per thread and tile
    constexpr int WAIT_STEADY = 0x0F70 | ((LPT * (S - 2)) & 0xF) | (((LPT * (S - 2)) >> 4) << 14);
    // This wave's LDS reads are complete (its loads in flight are left alone), then the workgroup
    // barrier: the waits above have made the awaited deposits of every wave visible before it.
    auto ring_barrier = [&]() {
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_s_barrier();
    };
    auto k_tile = [&](int kt, int cur, auto fetch_tag, auto more_tag, auto odd_tag) {
      constexpr bool fetch = decltype(fetch_tag)::value, more = decltype(more_tag)::value;
      constexpr int first = CHAINS == 4 && decltype(odd_tag)::value ? 2 : 0;       // this tile's first chain
      const int nxt = cur + 1 == S ? 0 : cur + 1;
      // The requests of tile kt+S-1 go out over the first two k steps: in one burst at the top they fill the queue of the address
      // unit, and a wave that waits for room in it issues no MFMA (one 64x64 wave per SIMD: 2048^3 f16 22.4 -> 21.1 us, 512 x 512 x
      // 32768 in 16 parts 28.2 -> 27.0; two 64x32 waves of 16x16 blocks 20.6 -> 20.0, 256x128 tiles 4096 x 2048 x 2048 33.9 -> 33.1).
#pragma unroll
      for (int ks = 0; ks < C::KSTEPS; ++ks) {
        if constexpr (fetch) {
          if (ks < 2) {
            const int dst = cur == 0 ? S - 1 : cur - 1;
            fetch_a((kt + S - 1) * BK, dst, ks, 2);
            fetch_b((kt + S - 1) * BK, dst, ks, 2);
          }
        }
        if (ks + 1 < C::KSTEPS) {
          read_frags(cur, ks + 1, (ks + 1) & 1);
        } else if constexpr (more) {
          if constexpr (fetch) __builtin_amdgcn_s_waitcnt(WAIT_STEADY);
          else __builtin_amdgcn_s_waitcnt(0x0F70);
          ring_barrier();
          read_frags(nxt, 0, 0);
        }
        if (ks + 1 < C::KSTEPS || more) mma(ks & 1, std::integral_constant<int, 1>{}, first + ks);
        else mma(ks & 1, std::integral_constant<int, 0>{}, first + ks);
        if (fetch && ks < 2) interleave_vmem(std::false_type{});
        else interleave();
      }
      return nxt;
    };
#pragma unroll
    for (int t = 0; t < S - 1; ++t)
      if (t < nk) {
        fetch_a(t * BK, t);
        fetch_b(t * BK, t);
      }
    if (nk >= S - 1) __builtin_amdgcn_s_waitcnt(WAIT_STEADY);      // S-1 tiles issued: tile 0 is the oldest
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    ring_barrier();
    read_frags(0, 0, 0);
    int cur = 0, kt = 0;
    if constexpr (CHAINS == 4) {
      for (; kt + S < nk; kt += 2) {
        cur = k_tile(kt, cur, std::true_type{}, std::true_type{}, std::false_type{});
        cur = k_tile(kt + 1, cur, std::true_type{}, std::true_type{}, std::true_type{});
      }
    }
    for (; kt + S - 1 < nk; ++kt) cur = k_tile(kt, cur, std::true_type{}, std::true_type{}, std::false_type{});
    for (; kt + 1 < nk; ++kt) cur = k_tile(kt, cur, std::false_type{}, std::true_type{}, std::true_type{});
    k_tile(kt, cur, std::false_type{}, std::false_type{}, std::true_type{});
  } else if constexpr (C::RSETS == 2) {
    // Register-staged, two k tiles of loads in flight: tile kt+2 is requested at the top of tile kt into the register
    // set that tile kt left, and tile kt+1 (requested a whole k tile earlier) goes to LDS at the end of kt.  With one
    // set a tile's loads had one tile's MFMA time to arrive, less than the memory latency for most tiles, and every
    // k tile waited.  Requests beyond K fall out of range and return at once.
    // Operands off the vector boundaries: the tiles that lie inside K are requested without a branch (`inner`).  Where the two
    // ways of fetch_loose meet, the compiler cannot count the requests behind the awaited ones and waits for all of them, the
    // tile just requested included: 2039 x 1511 x 1003 bf16 21.8 -> 20.3 us, 1523 x 471 x 1003 f16 transA 13.3 -> 11.5.
    auto k_tile = [&](int kt, auto set_tag, auto more_tag, auto inner_tag) {
      constexpr int set = decltype(set_tag)::value;
      constexpr bool more = decltype(more_tag)::value, inner = decltype(inner_tag)::value;
      const int cur = kt & 1, nxt = cur ^ 1;
#pragma unroll
      for (int ks = 0; ks < C::KSTEPS; ++ks) {
        if constexpr (more) {
          if (ks == 0 && inner) {
            fetch_inner((kt + 2) * BK, set);
          } else if (ks == 0) {
            fetch_a((kt + 2) * BK, 0, 0, 1, set);
            fetch_b((kt + 2) * BK, 0, 0, 1, set);
          }
        }
        if (ks + 1 < C::KSTEPS) {
          read_frags(cur, ks + 1, (ks + 1) & 1);
        } else if constexpr (more) {
          commit(nxt, set ^ 1);
          block_sync();
          read_frags(nxt, 0, 0);
        }
        mma(ks & 1, std::integral_constant<int, 0>{}, set * C::KSTEPS + ks);
        interleave();
      }
    };
    read_frags(0, 0, 0);
    int kt = 0;
    // (parts of fp32 tiles are a few k tiles long and lose 3 % to the larger kernel: 467 x 263 x 479 in six parts 10.9 -> 11.4 us)
    if constexpr (LOOSE_A && LOOSE_B && !(ES == 4 && SPLIT)) {
      constexpr int BEYOND = C::ASRC == A_KC && C::BSRC == B_KC ? 0 : EPC - 1;
      for (; tiles_inside(kt, 4, BK, BEYOND, Kx); kt += 2) {
        k_tile(kt, std::integral_constant<int, 0>{}, std::true_type{}, std::true_type{});
        k_tile(kt + 1, std::integral_constant<int, 1>{}, std::true_type{}, std::true_type{});
      }
    }
    for (; kt + 2 < nk; kt += 2) {
      k_tile(kt, std::integral_constant<int, 0>{}, std::true_type{}, std::false_type{});
      k_tile(kt + 1, std::integral_constant<int, 1>{}, std::true_type{}, std::false_type{});
    }
    const bool even = kt + 1 < nk;
    if (even) k_tile(kt++, std::integral_constant<int, 0>{}, std::true_type{}, std::false_type{});
    // (the last tile requests and deposits nothing: its set only tells the chains apart, which 16x16 fp32 products do by themselves: a copy of
    // the tile less, 512^3 fp32 6.46 -> 6.29 us)
    if (CHAINS > 1 && !(ES == 4 && MB == 16) && even) k_tile(kt, std::integral_constant<int, 1>{}, std::false_type{}, std::false_type{});
    else k_tile(kt, std::integral_constant<int, 0>{}, std::false_type{}, std::false_type{});
  } else if constexpr (PIPE) {
    // Whether a further k tile follows is a compile-time property of the loop body: the last k
    // tile is peeled.  With a run-time test the two paths would meet in front of the last k
    // step's MFMAs, where the compiler must then wait for the fragment reads issued after the
    // barrier (they are outstanding on one path only), which stalls every wave of the workgroup
    // at the same moment once per k tile.
    auto k_tile = [&](int kt, auto more_tag) {
      constexpr bool more = decltype(more_tag)::value;
      const int cur = kt & 1, nxt = cur ^ 1;
      // Wave tiles of eight and more MFMAs per k step issue the direct loads of the next tile over the
      // first two k steps, one between MFMAs, instead of in one burst at the top: with one such wave
      // per SIMD the burst is time no MFMA runs (256x256 tile of four 128x128 waves: 124 -> 116 us;
      // two 128x64 waves per SIMD gain 1 %; 64x64 wave tiles lose 1-8 % and keep the burst).
      constexpr int FS = (C::DIRECT && C::KSTEPS >= 4 && C::MBLK * C::NBLK >= 8) ? 2 : 1;
#pragma unroll
      for (int ks = 0; ks < C::KSTEPS; ++ks) {
        if constexpr (more) {
          if (ks < FS) {
            fetch_a((kt + 1) * BK, nxt, ks, FS);
            fetch_b((kt + 1) * BK, nxt, ks, FS);
          }
        }
        if (ks + 1 < C::KSTEPS) {
          read_frags(cur, ks + 1, (ks + 1) & 1);
        } else if constexpr (more) {
          commit(nxt);
          wait_deposits();
          block_sync();
          read_frags(nxt, 0, 0);
        }
        if (ks + 1 < C::KSTEPS || more) mma(ks & 1, std::integral_constant<int, 1>{});
        else mma(ks & 1, std::integral_constant<int, 0>{});
        if (FS > 1 && more && ks < FS) interleave_vmem(std::false_type{});
        else interleave();
      }
    };
    read_frags(0, 0, 0);
    for (int kt = 0; kt + 1 < nk; ++kt) k_tile(kt, std::true_type{});
    k_tile(nk - 1, std::false_type{});
  } else {
    for (int kt = 0; kt < nk; ++kt) {
      const bool more = kt + 1 < nk;
      const int cur = C::STAGES == 2 ? (kt & 1) : 0, nxt = C::STAGES == 2 ? (cur ^ 1) : 0;
      if (more) {
        if constexpr (!C::DIRECT || C::STAGES == 2) {
          fetch_a((kt + 1) * BK, nxt);
          fetch_b((kt + 1) * BK, nxt);
        }
      }
#pragma unroll
      for (int ks = 0; ks < C::KSTEPS; ++ks) {
        read_frags(cur, ks, 0);
        mma(0, std::integral_constant<int, 0>{});
      }
      if constexpr (C::STAGES == 1) {
        block_sync();                       // everyone is done reading the single buffer
        if constexpr (C::DIRECT) {
          if (more) {
            fetch_a((kt + 1) * BK, 0);
            fetch_b((kt + 1) * BK, 0);
          }
        }
      }
      if (more) commit(nxt);
      wait_deposits();
      block_sync();
    }
  }

  if constexpr (CHAINS > 1) {
    static_assert(C::RSETS == 2 || (C::RING_16 && C::KSTEPS == 2), "the loops that tell the chains apart");
#pragma unroll
    for (int half = CHAINS / 2; half >= 1; half /= 2)
#pragma unroll
      for (int n = 0; n < half; ++n)
#pragma unroll
        for (int i = 0; i < C::MBLK; ++i)
#pragma unroll
          for (int j = 0; j < C::NBLK; ++j)
#pragma unroll
            for (int v = 0; v < MF::NACC; ++v) chain(n, i, j)[v] += chain(n + half, i, j)[v];
  }

  // ---- split tile: this part's sums go to its slot, 16 bytes per lane and store, a wave's store one contiguous KiB;
  // split_reduce, launched behind this kernel, adds a tile's slots up and writes C.  (Written through: the lines
  // are on their way to memory while the other parts still multiply.)
  if (SPLIT && kparts > 1) {
    constexpr int NV = C::MBLK * C::NBLK * MF::NACC / 4;       // 16-byte groups per lane
    constexpr int SLOT_BYTES = BM * BN * 4;
    constexpr int WRITE_THROUGH = 16;                          // sc1
    const int64_t own = (int64_t)(wg - args.whole) * kparts + kpart;
    const __amdgpu_buffer_rsrc_t slot = __builtin_amdgcn_make_buffer_rsrc((void*)((char*)args.partials + own * (int64_t)SLOT_BYTES), 0,
                                                                          (uint32_t)SLOT_BYTES, RSRC_FLAGS);
#pragma unroll
    for (int g = 0; g < NV; ++g) {
      const int b = g / (MF::NACC / 4), q = g % (MF::NACC / 4);
      u32x4 v;
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = as_u32(acc[b / C::NBLK][b % C::NBLK][4 * q + x]);
      __builtin_amdgcn_raw_buffer_store_b128(v, slot, (uint32_t)((g * C::THREADS + tid) * 16), 0, WRITE_THROUGH);
      if (g % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    return;
  }

  // ---- batches of one or two k tiles.  Such a launch is bound by its stores, and an XCD starts the tiles of a batch
  // together: they all wait for that batch's operands to come from memory, behind the stores of the batch before.  So each
  // workgroup reads its share of the next batch once on the way to its own stores, and the XCD's L2 holds it when
  // its workgroups get there.  96 x 1024 x 1024 x 64 f16 on operands that are not in a cache: 88.9 -> 75 us.
  u32x4 ahead = {0u, 0u, 0u, 0u};
  if constexpr (AHEAD) {
    const int64_t at = ((int64_t)(wg - bidx * tiles_per_batch) * C::THREADS + tid) * 16;
    if (at < args.ahead_a + args.ahead_b && bidx + 1 < args.batch)
      ahead = *(const u32x4*)(at < args.ahead_a ? (const char*)args.A + (int64_t)(bidx + 1) * args.strideA * ES + at
                                               : (const char*)args.B + (int64_t)(bidx + 1) * args.strideB * ES + (at - args.ahead_a));
  }

  // ---- epilogue: C = alpha * acc + beta * C through a buffer descriptor that starts at this
  // tile's first element; rows outside the matrix fall out of its range, columns beyond it are
  // sent out of range explicitly (they would alias the next row).  Lane l of a 32x32 block holds
  // column l%32 and rows 8*(v/4) + 4*(l/32) + v%4 in acc[v] (16x16: column l%16, rows 4*(l/16) + v),
  // so one element store of a wave covers two whole 128-byte row segments of C (four 64-byte
  // ones for 16x16 blocks).  Accumulating the transposed block instead, for 16-byte vector stores
  // of four columns per lane, measured slower everywhere (32 rows x 32 bytes per instruction:
  // -3 % on the 4096^3 GEMM, -9 % on 8192x3072x768, -11 % on the store-bound K = 64 shapes).
  typedef typename C::OutT OutT;
  constexpr int OS = ElemSize<OutT>::value;
  char* Cb = (char*)args.C + (int64_t)bidx * args.strideC * OS;
  const float alpha = args.alpha, beta = args.beta;
  if constexpr (C::BSRC == B_CONV) {
    // output O[img][filter][p][q]: row = filter, col = (img, p, q)
    const int pq = args.cP * args.cQ;
#pragma unroll
    for (int bi = 0; bi < C::MBLK; ++bi)
#pragma unroll
      for (int bj = 0; bj < C::NBLK; ++bj) {
        const int col = n0 + block_col(bj) + frow;
        const int img = col / pq;
        const int64_t cbase = (int64_t)img * args.M * pq + (col - img * pq);
#pragma unroll
        for (int v = 0; v < MF::NACC; ++v) {
          const int r = (MB == 32) ? 8 * (v / 4) + 4 * fgrp + (v % 4) : 4 * fgrp + v;
          const int row = m0 + block_row(bi) + r;
          if (row < args.M && col < args.N) store_out<OutT>(Cb, cbase + (int64_t)row * pq, alpha * acc[bi][bj][v]);
        }
      }
  } else {
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Cb + ((int64_t)m0 * args.ldc + n0) * OS), 0,
        clamp_records(((int64_t)(rows_valid - 1) * args.ldc + cols_valid) * OS), RSRC_FLAGS);
    // C is stored with the write-through cache policy (sc1) unless the host says otherwise (args.through): every line goes to
    // memory at once instead of lying dirty in the L2 until it is evicted.  Measured against write-back: 10-15 % faster
    // on the store-bound shapes (96 x 1024 x 1024 x 64: 79 -> 70 us), 1-2 % on the 4096^3 and GPT-2 shapes, 0.5-2.5 %
    // slower on launches of many rounds of long tiles (8192^3, 65536 x 4096 x 1024), where a write-back L2
    // drains one tile's stores under the next tile's loop.  The policy is an immediate of the store
    // instruction: it is chosen where the beta path is, once per block.
    // One store costs an accumulator read, the scaling, one add and the store: the column part of the offset (or
    // an out-of-range one: adding a row offset below 2^31 keeps it out of range) is selected once per block column,
    // the row part is a per-lane base plus a multiple of the row pitch that is the same for the whole wave, and
    // whether C is read (beta) is decided once per block, not per element.
    const uint32_t pitch = (uint32_t)args.ldc * OS;
    auto store_block = [&](int bi, int bj, uint32_t lane_off, auto beta_tag, auto policy_tag) {
      constexpr bool with_beta = decltype(beta_tag)::value;
      constexpr int STORE_POLICY = decltype(policy_tag)::value;
#pragma unroll
      for (int v = 0; v < MF::NACC; ++v) {
        const int r = (MB == 32) ? 8 * (v / 4) + (v % 4) : v;      // row inside the block, less the lane group's 4 * fgrp
        const uint32_t off = lane_off + (uint32_t)r * pitch;
        float x = alpha * acc[bi][bj][v];
        if constexpr (OS == 4) {
          if constexpr (with_beta) x += beta * as_f32(__builtin_amdgcn_raw_buffer_load_b32(rc, off, 0, 0));
          __builtin_amdgcn_raw_buffer_store_b32(as_u32(x), rc, off, 0, STORE_POLICY);
        } else {
          if constexpr (with_beta) {
            const uint16_t old = __builtin_amdgcn_raw_buffer_load_b16(rc, off, 0, 0);
            x += beta * to_float<OutT>(&old, 0);
          }
          uint16_t bits;
          store_out<OutT>(&bits, 0, x);
          __builtin_amdgcn_raw_buffer_store_b16(bits, rc, off, 0, STORE_POLICY);
        }
      }
    };
    // 16-bit output in whole cache lines: 64 columns of a row are 128 bytes, but a block's row is 32 or 64, a lane holds one
    // column, and an element store moves two bytes a lane.  So a lane packs rows r and r + 1 of its column, trades with its
    // neighbour for the column pair of one of the two rows, and lane swaps bring the blocks side by side together: a store
    // then writes two whole lines, and half as many are issued.  It pays where a CU holds one workgroup, whose stores nothing
    // hides: pointwise 32 x 256 x 56 x 56 -> 512 stride 2, fp16, 19.2 -> 18.0 us; 8192 x 3072 x 768 bf16 on 16x16 blocks 49.6 -> 41.8.
    // Smaller wave tiles, whose stores run
    // under other waves' products, lose 1-3 % to the packing (96 x 1024 x 1024 x 64 fp16 57.9 -> 59.9, 8192 x 768 x 3072 40.4 ->
    // 40.9) and keep the element stores.
    // (Waves of 96 or 32 columns, pairs of 16x16 blocks: half lines.)  Rings of 16x16 blocks, whose element stores are quarter lines, gain
    // at every size: 2048^3 f16 128x128 21.3 -> 19.8 us, 8192 x 1024 x 4096 256x128 69.2 -> 62.2.
    constexpr bool PAIRS = OS == 2 && (C::ALTERNATE || C::RING_16 || (C::WM * C::WN >= 128 * 64 && C::WN % 64 == 0));
    constexpr bool HALF_LINES = C::WN % 64 != 0;
    if (PAIRS && args.paired) {
      if constexpr (PAIRS) {
        const uint32_t pick = (lane & 1) ? 0x03020706u : 0x05040100u;      // odd lanes: the second row
        auto pair_of = [&](int bi, int bj, int v) -> uint32_t {
          const uint32_t own = pack_out<OutT>(alpha * acc[bi][bj][v], alpha * acc[bi][bj][v + 1]);
          const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);      // quad_perm [1,0,3,2]
          return __builtin_amdgcn_perm(other, own, pick);
        };
        auto put = [&](uint32_t x, uint32_t off) {
          if (args.through) __builtin_amdgcn_raw_buffer_store_b32(x, rc, off, 0, 16);
          else __builtin_amdgcn_raw_buffer_store_b32(x, rc, off, 0, 0);
        };
        constexpr int GB = (HALF_LINES ? 32 : 64) / MB;                    // blocks in 64 (32) columns
#pragma unroll
        for (int bj = 0; bj < C::NBLK; bj += GB) {
          const int col = block_col(bj) + (lane % (GB * MB) & ~1);
          const uint32_t col_off = col < cols_valid ? (uint32_t)(col * OS) : OOB;
#pragma unroll
          for (int bi = 0; bi < C::MBLK; ++bi) {
            const uint32_t lane_off = col_off + (uint32_t)(block_row(bi) + (lane & 1) + (HALF_LINES ? 8 * (lane >> 5) : 0)) * pitch;
#pragma unroll
            for (int v = 0; v < MF::NACC; v += 2) {
              const int r = (MB == 32) ? 8 * (v / 4) + (v % 4) : v;        // rows r and r + 1 of lane group 0; groups are four rows apart
              if constexpr (MB == 32) {
                const auto q = __builtin_amdgcn_permlane32_swap(pair_of(bi, bj, v), pair_of(bi, bj + 1, v), false, false);
                put(q[0], lane_off + (uint32_t)r * pitch);
                put(q[1], lane_off + (uint32_t)(r + 4) * pitch);
              } else if constexpr (HALF_LINES) {
                const auto q = __builtin_amdgcn_permlane16_swap(pair_of(bi, bj, v), pair_of(bi, bj + 1, v), false, false);
                put(q[0], lane_off + (uint32_t)r * pitch);
                put(q[1], lane_off + (uint32_t)(r + 4) * pitch);
              } else {
                const auto a = __builtin_amdgcn_permlane16_swap(pair_of(bi, bj, v), pair_of(bi, bj + 1, v), false, false);
                const auto b = __builtin_amdgcn_permlane16_swap(pair_of(bi, bj + 2, v), pair_of(bi, bj + 3, v), false, false);
                const auto c = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
                const auto d = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
                put(c[0], lane_off + (uint32_t)r * pitch);
                put(d[0], lane_off + (uint32_t)(r + 4) * pitch);
                put(c[1], lane_off + (uint32_t)(r + 8) * pitch);
                put(d[1], lane_off + (uint32_t)(r + 12) * pitch);
              }
            }
          }
        }
      }
      return;
    }
    // fp32 output of 16x16 blocks: their rows are half lines, so two blocks side by side trade lane rows first and a store
    // writes two whole lines (rings: 8192 x 1024 x 4096 67.0 -> 65.6 us, 2048^3 20.8 -> 20.4)
    constexpr bool ROWS = (C::ALTERNATE || C::RING_16) && OS == 4;
    if (ROWS && beta == 0.f) {
      if constexpr (ROWS) {
        auto put = [&](uint32_t x, uint32_t off) {
          if (args.through) __builtin_amdgcn_raw_buffer_store_b32(x, rc, off, 0, 16);
          else __builtin_amdgcn_raw_buffer_store_b32(x, rc, off, 0, 0);
        };
#pragma unroll
        for (int bj = 0; bj < C::NBLK; bj += 2) {
          const int col = block_col(bj) + (lane & 31);
          const uint32_t col_off = col < cols_valid ? (uint32_t)(col * OS) : OOB;
#pragma unroll
          for (int bi = 0; bi < C::MBLK; ++bi) {
            const uint32_t lane_off = col_off + (uint32_t)(block_row(bi) + 8 * (lane >> 5)) * pitch;
#pragma unroll
            for (int v = 0; v < MF::NACC; ++v) {
              const auto q = __builtin_amdgcn_permlane16_swap(as_u32(alpha * acc[bi][bj][v]), as_u32(alpha * acc[bi][bj + 1][v]), false, false);
              put(q[0], lane_off + (uint32_t)v * pitch);
              put(q[1], lane_off + (uint32_t)(v + 4) * pitch);
            }
          }
        }
      }
      return;
    }
#pragma unroll
    for (int bj = 0; bj < C::NBLK; ++bj) {
      const int col = block_col(bj) + frow;
      const uint32_t col_off = col < cols_valid ? (uint32_t)(col * OS) : OOB;
#pragma unroll
      for (int bi = 0; bi < C::MBLK; ++bi) {
        const uint32_t lane_off = col_off + (uint32_t)(block_row(bi) + 4 * fgrp) * pitch;
        // (non-temporal where the next batch is read ahead, whose operands the caches are wanted for: 96 x 1024 x 1024 x 64,
        // outputs of 403 MB, 74.6 -> 61.8 us)
        constexpr std::integral_constant<int, AHEAD ? 18 : 16> write_through{};
        constexpr std::integral_constant<int, 0> write_back{};
        // (without the hint the fourth form cost the store-bound launches that do not use it 0.7 %)
        if (OS == 2 ? args.through != 0 : __builtin_expect(args.through && beta == 0.f, 1)) store_block(bi, bj, lane_off, std::false_type{}, write_through);
        else if (beta == 0.f) store_block(bi, bj, lane_off, std::false_type{}, write_back);
        else if (OS == 4 && args.through) store_block(bi, bj, lane_off, std::true_type{}, write_through);
        else store_block(bi, bj, lane_off, std::true_type{}, write_back);
      }
    }
  }
  if constexpr (AHEAD) asm volatile("" ::"v"(ahead));      // used by nothing: it lands before the wave ends
}

// ---- split-k: C = alpha * (sum of a tile's slots) + beta * C, one 16-byte group of a slot (four rows of one column) per
// thread.  The slots are added in part order, so the result does not depend on when a part finished.  Bound by the
// fp32 partial tiles it reads, (tiles - whole) * split * BM * BN * 4 bytes, spread over the whole chip.  An
// earlier form counted the parts of a tile in with atomics and let the last one add the slots up: that read them
// with one workgroup per tile, 16 of 256 CUs on 512 x 512 x 32768, and needed a launch of its own all the same,
// to clear the counters (that shape in 16 parts: 51.4 us, 38.7 us with this launch instead).
template <typename OutT>
__global__ __launch_bounds__(256) void split_reduce(const KernelArgs args, int bm, int bn, int wm, int wn, int mb) {
  const int threads = (bm / wm) * (bn / wn) * 64;          // of a workgroup of the contraction
  const int groups = bm * bn / 4;                          // 16-byte groups of a slot, a multiple of a block's 256
  const int blocks = groups >> 8;
  const int u = blockIdx.x / blocks, r = (blockIdx.x - u * blocks) * 256 + threadIdx.x;
  const int tiles_per_batch = args.tiles_m * args.tiles_n;
  const int wg = args.whole + u;
  if (wg >= tiles_per_batch * args.batch) return;
  // group r = g * threads + tid of the contraction's store: block g / (groups per block), four rows 8 * (g % ...) down
  const int g = r / threads, tid = r - g * threads;
  const int lane = tid & 63, wave = tid >> 6, waves_n = bn / wn, nblk = wn / mb;
  const int per_block = mb == 32 ? 4 : 1;
  const int b = g / per_block, q = g - b * per_block;
  const int row = (wave / waves_n) * wm + (b / nblk) * mb + 8 * q + 4 * (lane / mb);
  const int col = (wave % waves_n) * wn + (b % nblk) * mb + lane % mb;
  // A tile's slots through one descriptor: the loads that lie behind the last part read zero, at no cost.  All are in flight together, and
  // non-temporal, for nobody reads a slot again: with at most eight and without the hint 312 x 240 x 15552 in twelve parts of 64x64 tiles 14.3
  // us against 13.5, 560 x 408 x 17536 in twelve of 128x128 21.5 against 20.8, 128 x 128 x 4096 in sixteen of 32x32 7.1 against 6.9.
  const __amdgpu_buffer_rsrc_t slots = __builtin_amdgcn_make_buffer_rsrc((void*)((const f32x4*)args.partials + (int64_t)u * args.split * groups), 0,
                                                                        (uint32_t)(args.split * groups * 16), 0x00020000u);
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  auto add = [&](int o, auto n_tag) {
    constexpr int n = decltype(n_tag)::value;
    u32x4 v[n];
#pragma unroll
    for (int i = 0; i < n; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(slots, (uint32_t)(((o + i) * groups + r) * 16), 0, 2 /* nt */);
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
      for (int x = 0; x < 4; ++x) sum[x] += as_f32(v[i][x]);
  };
  if (args.split <= 2) add(0, std::integral_constant<int, 2>{});
  else if (args.split <= 4) add(0, std::integral_constant<int, 4>{});
  else if (args.split <= 8) add(0, std::integral_constant<int, 8>{});
  else add(0, std::integral_constant<int, 16>{});            // (split_allowed: there are no more)
  const int bidx = wg / tiles_per_batch;
  int tile_m, tile_n;
  tile_of(args, wg - bidx * tiles_per_batch, tile_m, tile_n);
  const int m = tile_m * bm + row, n = tile_n * bn + col;
  if (n >= args.N) return;
  const int64_t c0 = (int64_t)bidx * args.strideC + (int64_t)m * args.ldc + n;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    if (m + x >= args.M) break;
    float v = args.alpha * sum[x];
    if (args.beta != 0.f) v = fmaf(args.beta, to_float<OutT>(args.C, c0 + x * args.ldc), v);
    store_out<OutT>(args.C, c0 + x * args.ldc, v);
  }
}

}  // namespace gensor
