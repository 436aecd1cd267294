// Host-side declarations shared by the operator entry points and the constructor.
#pragma once
#include <stdint.h>

#include <vector>

#include "../../include/gensor.h"
#include "registry.hpp"

namespace gensor {

// GEMM view of a problem: C[M][N] += A[M][K] * B[K][N] per batch.
struct GemmView {
  int64_t M, N, K, batch;
  int64_t P, Q;          // convolution output extent
  int in_dtype, out_dtype, esize, osize;
  int bsrc;              // BSrc
  int asrc;              // ASrc: A stored [m][k] (A_KC) or [k][m] (A_MC, transA)
  int pointwise;         // convolution with a 1x1 filter and no padding, viewed as one GEMM per image
  // convolution geometry (zero otherwise)
  int64_t cn, cc, ch, cw, cr, cs, cstride, cpad;
};

// LDS plan of a patch-staged convolution instance for one problem.
struct ConvPlan {
  int a_pitch, patch_rows, stage_bytes, tile_px;
  int64_t in_bytes, w_bytes, out_bytes;
};
// Output pixels per workgroup of a patch-staged instance with a pixel tile of bn.  When output rows are
// shorter than the tile, a workgroup takes a whole number of them (its patch then has no partial rows):
// as many as fit, or fewer when that deals the tiles more evenly over `cus` compute units.  A tile's
// time is taken as 0.55 of a full tile's (MFMA work, filters, set-up: they do not shrink with the pixels)
// plus 0.45 in proportion to its pixels (patch loads, stores).
inline int64_t conv_tile_px(int64_t bn, int64_t N, int64_t Q, int64_t tiles_m, int64_t cus) {
  if (Q > bn) return bn;
  auto cost = [&](int64_t px) {
    const int64_t tiles = (N + px - 1) / px * tiles_m;
    return (double)((tiles + cus - 1) / cus) * (0.55 * (double)bn + 0.45 * (double)px);
  };
  int64_t best = bn / Q * Q;
  for (int64_t r = bn / Q - 1; r >= 1; --r)
    if (cost(r * Q) < cost(best)) best = r * Q;
  return best;
}
// The same for the row-staged convolution: input rows as they lie, `channels` of them per LDS stage.
struct ConvRowsPlan {
  int a_pitch, rows, row_pitch, channels, stage_bytes, tile_px;
  int64_t in_bytes, w_bytes, out_bytes;
};
// False if a row-staged instance with tile bm x bn cannot run the convolution in v.
bool conv_rows_plan(int bm, int bn, const GemmView& v, ConvRowsPlan* plan, int round_units = 0);
// False if instance d (a patch-staged convolution) cannot run the convolution in v.  round_units: the
// compute units the tiles are dealt over (0: the MI355X's).
bool conv_patch_plan(const InstanceDesc& d, const GemmView& v, ConvPlan* plan, int round_units = 0);

// A pointwise convolution (1x1 filter, no padding) is O[img] = W[k][c] * X[img][c][P*Q] with
// X the input sampled at the stride: a batched GEMM over the images with an n-contiguous B.
// VIEW_DEFAULT takes that view; with stride 2 and rows of whole 16-byte vectors the kernel
// samples the input while fetching it (B_NCS2), any other stride > 1 needs the input compacted
// into the workspace first (B_NC).  VIEW_PREPASS always compacts; VIEW_GENERAL gives the
// general implicit-GEMM view.  The three agree for every other operator.
enum ViewMode { VIEW_GENERAL = 0, VIEW_DEFAULT = 1, VIEW_PREPASS = 2 };
gensor_status gemm_view(const gensor_problem* p, GemmView* v, int mode = VIEW_DEFAULT);
void schedule_from_instance(const InstanceDesc& d, gensor_schedule* s);
bool instance_serves(const InstanceDesc& d, const GemmView& v);
const InstanceDesc* find_instance(const gensor_schedule* s, const GemmView& v);

// Workgroups and workspace of a split-k launch.
struct SplitPlan {
  int split;               // parts per split tile (1: nothing is split)
  int64_t whole;           // tiles computed by one workgroup each
  size_t bytes;            // partial tiles
};
// round_units: the compute units a round of tiles is dealt over (gensor_schedule::round_units; 0: the MI355X's).
SplitPlan split_plan(const InstanceDesc& d, const GemmView& v, int split, int round_units);
bool split_allowed(const InstanceDesc& d, const GemmView& v, int split);

// Does a launch of an instance whose wave groups alternate, with nothing split, cut C into tiles of 192 instead of 256 columns?
// A round of them takes 0.8 to 0.98 of a round of the wide ones, so: where they need no more rounds.  Wide and narrow, us, with
// rounds: 8192 x 3072 x 768 bf16 2/2 42.2 -> 38.8 (column-major B 42.1 -> 36.3), 2048 x 3072 x 4096 f16 1/1 73.6 -> 58.5, 4096 x 2560
// x 3072 1/1 62.6 -> 61.4; but 8192 x 4096 x 1024 bf16 2/3 57.3 -> 64.4, 4096^3 1/2 104.5 -> 135.7, 4096 x 4032 x 1024 1/2 34.8 -> 44.0.
inline bool narrow_tiles(const GemmView& v, int64_t compute_units) {
  const int64_t rows = (v.M + 255) / 256 * v.batch;
  const int64_t wide = (rows * ((v.N + 255) / 256) + compute_units - 1) / compute_units;
  const int64_t narrow = (rows * ((v.N + 191) / 192) + compute_units - 1) / compute_units;
  return narrow <= wide;
}

// The kernels address a workgroup tile with 32-bit offsets: can instance d, with leading dimensions `ld`?
struct LeadingDims { int64_t a, b, c; };
bool offsets_fit(const InstanceDesc& d, const GemmView& v, const LeadingDims& ld);

// gensor_construct with more inputs: whether the operands allow 16-byte vector accesses, the view (ViewMode) a
// pointwise convolution is taken in, and, where only tiles whose offsets reach are wanted, the leading dimensions.
// `ranked`: beside the best schedule, the best ones for less workspace than it needs, in order, down to one that needs none.
struct RankedSchedule { gensor_schedule schedule; size_t bytes; };
gensor_status construct_internal(const gensor_problem* p, const gensor_hw* hw, const gensor_construct_opts* opts,
                                 uint64_t seed, bool vec_ok, int view_mode, gensor_schedule* out, const LeadingDims* ld = nullptr,
                                 std::vector<RankedSchedule>* ranked = nullptr);

}  // namespace gensor
