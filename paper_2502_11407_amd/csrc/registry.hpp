// Table of the ahead-of-time compiled kernel instances: the finite part of the schedule
// lattice that exists as machine code.  Each entry is one point (tiles, virtual threads,
// staging mode, vector width) for one element type and operand source.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "conv_kernel.hpp"
#include "conv_rows_kernel.hpp"
#include "gemm_kernel.hpp"

namespace gensor {

struct InstanceDesc {
  int id;
  int in_dtype, out_dtype;              // gensor_dtype values
  int bm, bn, bk, wm, wn, mb, vm, vn;
  int bsrc;                             // BSrc
  int asrc;                             // ASrc
  int vec, stages, direct;
  int lds_bytes, threads, kg;           // kg: k consumed per fragment read (lds_bytes 0: set per problem)
  int units;                            // patch-staged convolution: transpose units per thread
  // 256x256 tiles whose wave groups alternate (Cfg::ALTERNATE); directly staged, they still take any K
  bool alternate() const { return direct && stages == 2 && mb == 16 && bm == 256 && bn == 256 && bk == 64; }
  // directly staged instances that take a K that is not a multiple of bk (Cfg::RING_16 are the others)
  bool any_k() const { return alternate() || (direct && stages > 2 && mb == 16); }
  bool conv_rows() const { return bsrc == B_CONV && direct && !vec; }      // the row-staged convolution
  hipError_t (*launch)(const KernelArgs&, hipStream_t);
  hipError_t (*launch_split)(const KernelArgs&, hipStream_t);   // the same instance with split tiles; null if not compiled
};

extern const InstanceDesc g_instances[];
extern const int g_num_instances;

// The dynamic-LDS limit of a kernel is a per-device attribute: set it once on every device
// the instance is launched on (one bit per device ordinal; thread-safe, setting twice is harmless).
template <typename K>
hipError_t allow_dynamic_lds(K kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  done.fetch_or(bit, std::memory_order_release);
  return hipSuccess;
}

// Does a launch keep Cfg::DEEP_CHAINS sums per output?  They take 0.1-0.5 us to clear and to add up, and registers.
// Rings: from 24 k tiles (whole tiles of fewer never stood for parts; with four sums 1782 x 2048 x 512 took 7.4 us instead of 7.0, 1280 x 1408 x
//   1600 13.4 instead of 13.1), parts from twelve with two sums (512 x 2048 x 4600 transA, six parts where there were eight) and from
//   sixteen with four.
// Any-alignment 16-bit 64x64 tiles: parts from seven, whole ones from sixteen (22 of 450 x 64 x 450 6.5 us instead of 6.2), as long as the three
//   workgroups a compute unit then holds, instead of four, are all there are (67 of 919 x 64 x 919, 1005 workgroups, 31.0 us instead of 29.3).
//   128x64 tiles: whole ones from 24, one to a unit (56 of 970 x 64 x 970, 448 workgroups, 28.9 us instead of 23.3), which stood for two parts.
// Any-alignment fp32 64x64 tiles: whole ones that stand for three 64x32 tiles of eight sums to a unit.
template <typename C, bool SPLIT>
bool more_sums(const KernelArgs& a, unsigned workgroups) {
  const int depth = (a.K + C::BK - 1) / C::BK / (SPLIT && a.whole == 0 ? a.split : 1);
  if (C::DIRECT) return depth >= (!SPLIT ? 24 : C::DEEP_CHAINS == 2 ? 12 : 16);
  if (C::ES == 4) return !SPLIT && depth >= 3 && workgroups > 256 && workgroups <= 384;
  if (C::BM == 128) return !SPLIT && depth >= 24 && workgroups <= 256;
  return depth >= (SPLIT ? 7 : 16) && workgroups <= 3 * 256;
}

template <typename C, bool SPLIT = false, bool AHEAD = false, bool MORE_SUMS = false>
hipError_t launch_instance(const KernelArgs& a, hipStream_t st) {
  if constexpr (C::HAS_AHEAD && !SPLIT && !AHEAD) {
    if (a.ahead_a + a.ahead_b > 0) return launch_instance<C, false, true>(a, st);
  }
  if constexpr (C::HAS_NARROW && !SPLIT) {
    if (a.narrow) return launch_instance<NarrowCfg<C>>(a, st);
  }
  // one workgroup per whole tile and, in a split launch, a.split per tile behind them
  const unsigned tiles = (unsigned)a.tiles_m * (unsigned)a.tiles_n * (unsigned)a.batch;
  const unsigned grid = SPLIT ? (unsigned)a.whole + (tiles - (unsigned)a.whole) * (unsigned)a.split : tiles;
  if constexpr (C::DEEP_CHAINS != C::CHAINS && !MORE_SUMS) {
    if (more_sums<C, SPLIT>(a, grid)) return launch_instance<C, SPLIT, AHEAD, true>(a, st);
  }
  static std::atomic<uint64_t> done{0};
  hipError_t e = allow_dynamic_lds(contraction_kernel<C, SPLIT, AHEAD, MORE_SUMS>, C::LDS_BYTES, done);
  if (e != hipSuccess) return e;
  const int lds_bytes = C::ALTERNATE || a.lds_stages >= C::STAGES ? C::LDS_BYTES : C::STAGE_BYTES * a.lds_stages;
  hipLaunchKernelGGL((contraction_kernel<C, SPLIT, AHEAD, MORE_SUMS>), dim3(grid), dim3(C::THREADS), lds_bytes, st, a);
  return hipGetLastError();
}

// row-staged convolution: the LDS size depends on the problem
template <typename C, bool ONE_CHUNK>
hipError_t launch_conv_rows_as(const KernelArgs& a, hipStream_t st) {
  static std::atomic<uint64_t> done{0};
  hipError_t e = allow_dynamic_lds(conv_rows_kernel<C, ONE_CHUNK>, 160 * 1024, done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((conv_rows_kernel<C, ONE_CHUNK>), dim3((unsigned)a.tiles_m * (unsigned)a.tiles_n), dim3(C::THREADS), a.cStageBytes, st, a);
  return hipGetLastError();
}
template <typename C>
hipError_t launch_conv_rows(const KernelArgs& a, hipStream_t st) {
  return a.cS <= C::EPC ? launch_conv_rows_as<C, true>(a, st) : launch_conv_rows_as<C, false>(a, st);
}

// patch-staged convolution: the LDS size depends on the problem (a.cStageBytes per LDS stage
// plus, unless the filter is 1x1 or 3x3, one raw filter region of BM * R*S*BKC elements).
template <typename C, int FMODE, bool THROUGH, bool TAIL>
hipError_t launch_conv_tail(const KernelArgs& a, hipStream_t st, int raw_bytes) {
  static std::atomic<uint64_t> done{0};
  hipError_t e = allow_dynamic_lds(conv_patch_kernel<C, FMODE, THROUGH, TAIL>, 160 * 1024, done);
  if (e != hipSuccess) return e;
  const unsigned grid = (unsigned)a.tiles_m * (unsigned)a.tiles_n;
  hipLaunchKernelGGL((conv_patch_kernel<C, FMODE, THROUGH, TAIL>), dim3(grid), dim3(C::THREADS), C::LSTAGES * a.cStageBytes + raw_bytes, st, a);
  return hipGetLastError();
}

// Moving back the vectors that would run past the input's end is compiled only into the launches that can need it:
// 16-bit elements and an odd row length (any other vector that runs past the end starts on a dword boundary and
// the buffer's range check returns its valid part).
template <typename C, int FMODE, bool THROUGH>
hipError_t launch_conv_route(const KernelArgs& a, hipStream_t st, int raw_bytes) {
  if constexpr (C::ES == 2) {
    if (a.cW & 1) return launch_conv_tail<C, FMODE, THROUGH, true>(a, st, raw_bytes);
  }
  return launch_conv_tail<C, FMODE, THROUGH, false>(a, st, raw_bytes);
}

// The output is stored write-through when the reduction is shallow (the stores are then a large share of
// the launch), write-back otherwise.
template <typename C, bool THROUGH>
hipError_t launch_conv_policy(const KernelArgs& a, hipStream_t st) {
  const int rs = a.cR * a.cS;
  if (rs == 9) return launch_conv_route<C, 2, THROUGH>(a, st, 0);       // 3x3 and 1x1 reorder their filters in registers
  if (rs == 1) return launch_conv_route<C, 1, THROUGH>(a, st, 0);
  return launch_conv_route<C, 0, THROUGH>(a, st, C::BM * rs * C::BKC * C::ES);      // the others through a raw LDS region
}

template <typename C>
hipError_t launch_conv_instance(const KernelArgs& a, hipStream_t st) {
  return a.K <= 1024 ? launch_conv_policy<C, true>(a, st) : launch_conv_policy<C, false>(a, st);
}

}  // namespace gensor
