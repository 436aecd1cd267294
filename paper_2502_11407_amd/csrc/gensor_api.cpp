// C ABI of the operators: argument validation, GEMM view of each operator, lookup of the
// kernel instance a schedule names, and the launch.  No device memory is allocated here.
#include <hip/hip_runtime.h>

#include <array>
#include <cstring>
#include <map>
#include <mutex>
#include <utility>

#include "../../include/gensor.h"
#include "host_common.hpp"
#include "registry.hpp"

using namespace gensor;

extern "C" const char* gensor_status_string(gensor_status st) {
  switch (st) {
    case GENSOR_OK: return "ok";
    case GENSOR_ERR_INVALID_ARG: return "invalid argument";
    case GENSOR_ERR_UNSUPPORTED: return "unsupported combination";
    case GENSOR_ERR_NO_SCHEDULE: return "no feasible schedule / schedule does not match a compiled instance";
    case GENSOR_ERR_WORKSPACE: return "workspace too small";
    case GENSOR_ERR_DEVICE: return "HIP launch error";
  }
  return "unknown status";
}

extern "C" int32_t gensor_num_instances(void) { return g_num_instances; }

namespace gensor {

static bool valid_dtype(int d) { return d == GENSOR_F32 || d == GENSOR_F16 || d == GENSOR_BF16; }

gensor_status gemm_view(const gensor_problem* p, GemmView* v, int mode) {
  if (!p || !v) return GENSOR_ERR_INVALID_ARG;
  if (!valid_dtype(p->in_dtype) || !valid_dtype(p->out_dtype)) return GENSOR_ERR_INVALID_ARG;
  if (p->out_dtype != GENSOR_F32 && p->out_dtype != p->in_dtype) return GENSOR_ERR_UNSUPPORTED;
  std::memset(v, 0, sizeof(*v));
  v->in_dtype = p->in_dtype;
  v->out_dtype = p->out_dtype;
  v->esize = p->in_dtype == GENSOR_F32 ? 4 : 2;
  v->osize = p->out_dtype == GENSOR_F32 ? 4 : 2;
  if (p->op == GENSOR_OP_GEMM || p->op == GENSOR_OP_BMM) {
    if (p->M <= 0 || p->N <= 0 || p->K <= 0) return GENSOR_ERR_INVALID_ARG;
    if (p->op == GENSOR_OP_BMM && p->batch <= 0) return GENSOR_ERR_INVALID_ARG;
    if ((p->transA != 0 && p->transA != 1) || (p->transB != 0 && p->transB != 1)) return GENSOR_ERR_INVALID_ARG;
    v->M = p->M; v->N = p->N; v->K = p->K;
    v->batch = p->op == GENSOR_OP_BMM ? p->batch : 1;
    v->bsrc = p->transB ? B_KC : B_NC;
    v->asrc = p->transA ? A_MC : A_KC;
  } else if (p->op == GENSOR_OP_CONV2D) {
    if (p->n <= 0 || p->c <= 0 || p->h <= 0 || p->w <= 0 || p->k <= 0 || p->r <= 0 || p->s <= 0) return GENSOR_ERR_INVALID_ARG;
    if (p->stride <= 0 || p->pad < 0) return GENSOR_ERR_INVALID_ARG;
    if (p->h + 2 * p->pad < p->r || p->w + 2 * p->pad < p->s) return GENSOR_ERR_INVALID_ARG;
    v->P = (p->h + 2 * p->pad - p->r) / p->stride + 1;
    v->Q = (p->w + 2 * p->pad - p->s) / p->stride + 1;
    v->M = p->k;
    v->N = p->n * v->P * v->Q;
    v->K = p->c * p->r * p->s;
    v->batch = 1;
    v->bsrc = B_CONV;
    v->cn = p->n; v->cc = p->c; v->ch = p->h; v->cw = p->w; v->cr = p->r; v->cs = p->s;
    v->cstride = p->stride; v->cpad = p->pad;
    if (mode != VIEW_GENERAL && p->r == 1 && p->s == 1 && p->pad == 0) {
      v->pointwise = 1;
      v->N = v->P * v->Q;
      v->K = p->c;
      v->batch = p->n;
      // stride 2 on rows that are whole 16-byte vectors: sampled while fetched, no pre-pass
      v->bsrc = (mode == VIEW_DEFAULT && p->stride == 2 && p->w % (16 / v->esize) == 0) ? B_NCS2 : B_NC;
    }
  } else {
    return GENSOR_ERR_INVALID_ARG;
  }
  if (v->M > INT32_MAX || v->N > INT32_MAX || v->K > INT32_MAX || v->batch > INT32_MAX) return GENSOR_ERR_UNSUPPORTED;
  return GENSOR_OK;
}

void schedule_from_instance(const InstanceDesc& d, gensor_schedule* s) {
  std::memset(s, 0, sizeof(*s));
  s->version = GENSOR_SCHEDULE_VERSION;
  s->kernel_id = d.id;
  s->tile[GENSOR_DIM_M][0] = d.bm; s->tile[GENSOR_DIM_N][0] = d.bn; s->tile[GENSOR_DIM_K][0] = d.bk;
  s->tile[GENSOR_DIM_M][1] = d.wm; s->tile[GENSOR_DIM_N][1] = d.wn; s->tile[GENSOR_DIM_K][1] = d.kg;
  s->vthread[0] = d.vm; s->vthread[1] = d.vn;
  s->tile[GENSOR_DIM_M][2] = d.wm / d.vm; s->tile[GENSOR_DIM_N][2] = d.wn / d.vn; s->tile[GENSOR_DIM_K][2] = d.kg;
  s->stages = d.stages;
  s->unroll = d.bk / d.kg;
  s->vec_bytes = d.vec ? 16 : (d.in_dtype == GENSOR_F32 ? 4 : 2);
  s->direct_lds = d.direct;
  s->split_k = 1;
  s->wg_remap = 4;
}

bool conv_patch_plan(const InstanceDesc& d, const GemmView& v, ConvPlan* plan, int round_units) {
  const int64_t lim = 0x7fffffffll;
  const int epc = 16 / v.esize;
  const int64_t rs = v.cr * v.cs;
  if (rs > 9 || v.cc % epc != 0) return false;
  ConvPlan pl;
  pl.in_bytes = v.cn * v.cc * v.ch * v.cw * v.esize;
  pl.w_bytes = v.M * v.K * v.esize;
  pl.out_bytes = v.M * v.N * v.osize;
  if (pl.in_bytes >= lim || pl.w_bytes >= lim || pl.out_bytes >= lim) return false;
  // filter tile: [bm][rs * bkc] with a row pitch of an odd number of 16-byte chunks
  int64_t p16 = rs * d.bk * v.esize / 16;
  if (p16 % 2 == 0) ++p16;
  pl.a_pitch = (int)(p16 * 16);
  if ((int64_t)d.bm * pl.a_pitch >= (1 << 20)) return false;
  // patch rows: the most stacked padded input rows any pixel tile touches
  const int64_t hp = v.ch + 2 * v.cpad, pw = v.cw + 2 * v.cpad;
  const int64_t cus = round_units > 0 ? round_units : gensor_hw_mi355x()->compute_units;
  const int64_t px = conv_tile_px(d.bn, v.N, v.Q, (v.M + d.bm - 1) / d.bm, cus);
  pl.tile_px = (int)px;
  int64_t rows = 0;
  for (int64_t n0 = 0; n0 < v.N; n0 += px) {
    const int64_t n1 = (n0 + px < v.N ? n0 + px : v.N) - 1;
    const int64_t g0 = n0 / v.Q, g1 = n1 / v.Q;
    const int64_t r0 = (g0 / v.P) * hp + (g0 % v.P) * v.cstride;
    const int64_t r1 = (g1 / v.P) * hp + (g1 % v.P) * v.cstride + v.cr - 1;
    if (r1 - r0 + 1 > rows) rows = r1 - r0 + 1;
  }
  pl.patch_rows = (int)rows;
  const int slot = d.bk * v.esize + 16;
  const int64_t stage = (int64_t)d.bm * pl.a_pitch + rows * pw * slot;
  const int64_t raw = (rs == 1 || rs == 9) ? 0 : (int64_t)d.bm * rs * d.bk * v.esize;      // raw filter runs, one buffer
  if (d.stages * stage + raw > 160 * 1024) return false;
  pl.stage_bytes = (int)stage;
  const int64_t units = rows * ((v.cw + epc - 1) / epc) * (d.bk / epc);
  if (units > (int64_t)d.units * d.threads) return false;
  if (plan) *plan = pl;
  return true;
}

bool conv_rows_plan(int bm, int bn, const GemmView& v, ConvRowsPlan* plan, int round_units) {
  const int64_t lim = 0x7fffffffll - 64;      // 32-bit offsets, with room for the descriptor's alignment
  const int64_t epc = 16 / v.esize;
  ConvRowsPlan pl;
  pl.in_bytes = v.cn * v.cc * v.ch * v.cw * v.esize;
  pl.w_bytes = v.cc * v.cr * v.cs * v.M * v.esize;
  pl.out_bytes = v.M * v.cn * v.P * v.Q * v.osize;
  if (pl.in_bytes >= lim || pl.w_bytes >= lim || pl.out_bytes >= lim) return false;
  const int64_t hp = v.ch + 2 * v.cpad;
  const int64_t cus = round_units > 0 ? round_units : gensor_hw_mi355x()->compute_units;
  const int64_t N = v.cn * v.P * v.Q;
  if (hp * v.cn > lim || v.cw + 2 * v.cpad > lim / 64) return false;
  const int64_t px = conv_tile_px(bn, N, v.Q, (v.M + bm - 1) / bm, cus);
  pl.tile_px = (int)px;
  // the most stacked padded input rows a pixel tile can touch: it covers out_rows output rows (one more than it fills
  // unless it is whole rows) and starts at any row of an image
  int64_t out_rows = px % v.Q == 0 ? px / v.Q : (px + v.Q - 2) / v.Q + 1;
  if (out_rows > v.cn * v.P) out_rows = v.cn * v.P;
  // (its last row is `images` images and `more` rows further on, or one image more where it starts among the last `more`
  // rows of an image and another follows; in closed form, for the plan is made in every call and an image may have any number of rows)
  const int64_t images = (out_rows - 1) / v.P, more = (out_rows - 1) % v.P;
  int64_t rows = images * hp + more * v.cstride + v.cr;
  if (more > 0 && images + 1 < v.cn && (images + 1) * hp + (more - v.P) * v.cstride + v.cr > rows)
    rows = (images + 1) * hp + (more - v.P) * v.cstride + v.cr;
  pl.rows = (int)rows;
  const int64_t xo = (v.cpad + epc - 1) / epc * epc;
  const int64_t right = (v.cw + v.cpad + epc - 1) / epc * epc;
  pl.row_pitch = (int)((xo + right) * v.esize);
  const int64_t sc = (v.cs + epc - 1) / epc;
  // Channels per stage: as many as fit an equal share of the LDS for every workgroup of a CU, up to three of them (a
  // stage is a round trip to memory that only the CU's other workgroups cover), at least one
  const int64_t wgs = ((v.M + bm - 1) / bm * ((N + px - 1) / px) + cus - 1) / cus;
  const int64_t share = 160 * 1024 / (wgs < 3 ? wgs : 3) / 16 * 16;
  auto bytes = [&](int64_t ch) {
    int64_t chunks = (ch * v.cr * sc + 1) / 2 * 2 + 1;        // an odd number of 16-byte chunks
    // (the last chunk of a window's row may reach 15 bytes beyond the last row, and its fifth dword four more: read and
    // cleared, never used)
    return std::make_pair((int64_t)bm * chunks * 16, ch * rows * pl.row_pitch + (sc * 16 + 32));
  };
  auto total = [&](int64_t ch) { auto b = bytes(ch); return (b.first + b.second + 15) / 16 * 16; };
  int64_t ch = v.cc;
  while (ch > 1 && total(ch) > share) ch = (ch + 1) / 2;
  // the kernel divides unit numbers by multiplying with a reciprocal: number times divisor stay below 2^31
  const int64_t segs = (v.cw + epc - 1) / epc, chunks = ch * v.cr * sc + 1, slack = 10 * 256;
  if (total(ch) > 160 * 1024 || sc > 15 || (bm * chunks + slack) * chunks > lim || (ch * rows * segs + slack) * (segs > rows ? segs : rows) > lim ||
      (hp * v.cn + rows) * hp > lim || (v.Q + bn) * v.Q > lim || (v.P + bn) * v.P > lim)
    return false;
  pl.channels = (int)ch;
  pl.a_pitch = (int)(bytes(ch).first / bm);
  pl.stage_bytes = (int)total(ch);
  if (plan) *plan = pl;
  return true;
}

bool instance_serves(const InstanceDesc& d, const GemmView& v) {
  if (d.in_dtype != v.in_dtype || d.out_dtype != v.out_dtype || d.bsrc != v.bsrc || d.asrc != v.asrc) return false;
  if (d.units) return conv_patch_plan(d, v, nullptr);
  if (d.conv_rows()) return conv_rows_plan(d.bm, d.bn, v, nullptr);
  // the kernels number k, and the requests that run to the end of the last k tile, in 32 bits
  return v.bsrc == B_CONV || v.K <= INT32_MAX - d.bk + 1;
}

// Does instance d realise schedule s (same lattice point)?
static bool instance_matches(const InstanceDesc& d, const gensor_schedule* s) {
  return d.bm == s->tile[0][0] && d.bn == s->tile[1][0] && d.bk == s->tile[2][0] && d.wm == s->tile[0][1] &&
         d.wn == s->tile[1][1] && d.kg == s->tile[2][1] && d.vm == s->vthread[0] && d.vn == s->vthread[1] &&
         d.stages == s->stages && d.direct == s->direct_lds && (d.vec ? 16 : -1) == (s->vec_bytes == 16 ? 16 : -1);
}

const InstanceDesc* find_instance(const gensor_schedule* s, const GemmView& v) {
  if (!s || s->version != GENSOR_SCHEDULE_VERSION) return nullptr;
  if (s->kernel_id >= 0 && s->kernel_id < g_num_instances) {
    const InstanceDesc& d = g_instances[s->kernel_id];
    if (instance_serves(d, v) && instance_matches(d, s)) return &d;
  }
  for (int i = 0; i < g_num_instances; ++i)
    if (instance_serves(g_instances[i], v) && instance_matches(g_instances[i], s)) return &g_instances[i];
  return nullptr;
}

bool offsets_fit(const InstanceDesc& d, const GemmView& v, const LeadingDims& ld) {
  const int64_t lim = 0x7fffffffll;
  if (v.asrc == A_KC && (int64_t)(d.bm + 1) * ld.a * v.esize >= lim) return false;
  if (v.asrc == A_MC && ((int64_t)(d.bk + 1) * ld.a + d.bm) * v.esize >= lim) return false;
  // (the convolution epilogues address the output with 64-bit indices and never use ldc)
  if (v.bsrc != B_CONV && (int64_t)(d.bm + 1) * ld.c * v.osize >= lim) return false;
  if (v.bsrc == B_KC && (int64_t)(d.bn + 1) * ld.b * v.esize >= lim) return false;
  if ((v.bsrc == B_NC || v.bsrc == B_NCS2) && ((int64_t)(d.bk + 1) * ld.b + d.bn) * v.esize >= lim) return false;
  return true;
}

// Can the 16-byte vector path be used?  (k-contiguous operands need K and their leading
// dimension to be whole chunks; the n-contiguous operand needs N and ldb to be.)
bool vector_ok(const GemmView& v, const void* A, int64_t lda, int64_t strideA, const void* B, int64_t ldb, int64_t strideB) {
  const int epc = 16 / v.esize;
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  if (!al(A) || lda % epc || strideA % epc || (v.asrc == A_KC ? v.K : v.M) % epc) return false;
  if (v.asrc == A_MC && v.bsrc == B_KC && v.K % epc) return false;
  if (v.bsrc == B_KC) return al(B) && ldb % epc == 0 && strideB % epc == 0;
  if (v.bsrc == B_NC || v.bsrc == B_NCS2) return al(B) && ldb % epc == 0 && strideB % epc == 0 && v.N % epc == 0;
  return al(B);  // convolution: the gather is element-wise; the patch path reads 16-byte vectors
}

}  // namespace gensor

extern "C" gensor_status gensor_instance_schedule(int32_t id, const gensor_problem* p, gensor_schedule* out) {
  if (!p || !out || id < 0 || id >= g_num_instances) return GENSOR_ERR_INVALID_ARG;
  GemmView v;
  gensor_status st = gemm_view(p, &v);
  if (st != GENSOR_OK) return st;
  if (!instance_serves(g_instances[id], v)) return GENSOR_ERR_UNSUPPORTED;
  schedule_from_instance(g_instances[id], out);
  return GENSOR_OK;
}

namespace gensor {
// Bytes of the compacted input of a strided pointwise convolution (0: the input is used as it is).
static size_t pointwise_workspace(const GemmView& v) {
  return v.pointwise && v.cstride > 1 && v.bsrc != B_NCS2 ? (size_t)(v.batch * v.K * v.N * v.esize) : 0;
}

// Split-k plan of instance d on view v with split factor `split`: the tiles that do not fill a whole
// round of compute units (all of them when there are fewer tiles than units) are computed by `split`
// workgroups each.  whole = tiles left unsplit; a plan with whole == tiles splits nothing.
SplitPlan split_plan(const InstanceDesc& d, const GemmView& v, int split, int round_units) {
  SplitPlan pl;
  const int64_t tiles = ((v.M + d.bm - 1) / d.bm) * ((v.N + d.bn - 1) / d.bn) * v.batch;
  const int64_t cus = round_units > 0 ? round_units : gensor_hw_mi355x()->compute_units;
  pl.whole = split > 1 ? tiles / cus * cus : tiles;
  pl.split = pl.whole == tiles ? 1 : split;
  pl.bytes = pl.split > 1 ? (size_t)((tiles - pl.whole) * pl.split * (int64_t)d.bm * d.bn * 4) : 0;
  return pl;
}

// Can the instance run a split tile?  It was compiled with the split path (operands fetched plainly, no
// gather, no sampling) and every part gets at least one k tile.
bool split_allowed(const InstanceDesc& d, const GemmView& v, int split) {
  if (split == 1) return true;
  if (split < 1 || split > 16 || !d.launch_split || (v.bsrc != B_KC && v.bsrc != B_NC)) return false;
  return (v.K + d.bk - 1) / d.bk >= split;
}

// The second launch of a split contraction (512 x 512 x 32768 f16 in 16 parts: 5 of the pair's 29 us).
static hipError_t launch_split_reduce(const InstanceDesc& d, const KernelArgs& a, hipStream_t st) {
  const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n * a.batch - a.whole;
  const int64_t blocks = (tiles * (d.bm * d.bn / 4) + 255) / 256;
  if (blocks > INT32_MAX) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)blocks), block(256);
  switch (d.out_dtype) {
    case GENSOR_F32: hipLaunchKernelGGL(split_reduce<f32_t>, grid, block, 0, st, a, d.bm, d.bn, d.wm, d.wn, d.mb); break;
    case GENSOR_F16: hipLaunchKernelGGL(split_reduce<f16_t>, grid, block, 0, st, a, d.bm, d.bn, d.wm, d.wn, d.mb); break;
    default: hipLaunchKernelGGL(split_reduce<bf16_t>, grid, block, 0, st, a, d.bm, d.bn, d.wm, d.wn, d.mb); break;
  }
  return hipGetLastError();
}
}  // namespace gensor

// Only a strided pointwise convolution run as a batched GEMM through the compaction pre-pass
// needs a workspace (the compacted copy of its input).
extern "C" size_t gensor_workspace_bytes(const gensor_schedule* s, const gensor_problem* p) {
  GemmView v, w;
  if (p && s && (p->op == GENSOR_OP_GEMM || p->op == GENSOR_OP_BMM)) {
    // a split-k schedule: one fp32 tile per part of every split tile
    if (s->split_k <= 1 || gemm_view(p, &v) != GENSOR_OK) return 0;
    const InstanceDesc* d = find_instance(s, v);
    return d && split_allowed(*d, v, s->split_k) ? split_plan(*d, v, s->split_k, s->round_units).bytes : 0;
  }
  if (!p || p->op != GENSOR_OP_CONV2D || gemm_view(p, &v) != GENSOR_OK || gemm_view(p, &w, VIEW_PREPASS) != GENSOR_OK) return 0;
  const size_t need_pw = pointwise_workspace(w);
  if (!s) return need_pw;                    // what any schedule the library may construct can ask for
  if (v.pointwise && find_instance(s, v)) return pointwise_workspace(v);
  if (w.pointwise && find_instance(s, w)) return need_pw;
  return 0;
}

// ------------------------------------------------------------------------------------
// schedule == NULL: construct once per (problem, alignment class) and remember what the ranking found for any workspace.
// ------------------------------------------------------------------------------------
namespace {
std::mutex g_memo_mutex;
std::map<std::array<int64_t, 17>, std::vector<RankedSchedule>> g_memo;
const size_t kMemoLimit = 4096;      // shapes remembered; a full memo is emptied (a shape seen again is constructed again)

// The largest leading dimension that the same tiles reach: tiles of 2^n rows (or k rows, with `beside` elements more in one) tell no
// two of them apart, so one construction serves all.
int64_t same_reach(int64_t ld, int esize, int64_t beside) {
  for (int rows = 256; rows >= 16; rows /= 2) {
    const int64_t most = ((0x7fffffffll - 1) / esize - beside) / (rows + 1);
    if (ld <= most) return most;
  }
  return ld;
}

// The best schedule that needs at most `room` bytes of workspace.
gensor_status memoised_schedule(const gensor_problem* p, bool vec_ok, int view_mode, size_t room, gensor_schedule* out,
                                const LeadingDims* ld = nullptr) {
  const bool conv = p->op == GENSOR_OP_CONV2D;
  const std::array<int64_t, 17> key = {p->op, p->in_dtype, p->out_dtype, p->transB + 2 * p->transA, (vec_ok ? 1 : 0) + 2 * view_mode,
                                       conv ? p->n : p->batch, conv ? p->c : p->M, conv ? p->h : p->N, conv ? p->w : p->K,
                                       conv ? p->k : 0, conv ? p->r : 0, conv ? p->s : 0, conv ? p->stride : 0, conv ? p->pad : 0,
                                       ld ? ld->a : 0, ld ? ld->b : 0, ld ? ld->c : 0};
  std::lock_guard<std::mutex> lock(g_memo_mutex);
  auto it = g_memo.find(key);
  if (it == g_memo.end()) {
    std::vector<RankedSchedule> ranked;
    gensor_status st = construct_internal(p, nullptr, nullptr, 0, vec_ok, view_mode, out, ld, &ranked);
    if (st != GENSOR_OK) return st;
    if (g_memo.size() >= kMemoLimit) g_memo.clear();
    it = g_memo.emplace(key, std::move(ranked)).first;
  }
  for (const RankedSchedule& r : it->second)
    if (r.bytes <= room) { *out = r.schedule; return GENSOR_OK; }
  return GENSOR_ERR_NO_SCHEDULE;
}

gensor_status run(const gensor_schedule* s, const gensor_problem* p, const GemmView& v, float alpha,
                  const void* A, int64_t lda, int64_t strideA, const void* B, int64_t ldb, int64_t strideB,
                  float beta, void* C, int64_t ldc, int64_t strideC, void* workspace, size_t workspace_bytes, void* stream) {
  const bool vec_ok = vector_ok(v, A, lda, strideA, B, ldb, strideB);
  const bool ws_aligned = workspace && (reinterpret_cast<uintptr_t>(workspace) & 255u) == 0;
  gensor_schedule local;
  const LeadingDims ld = {lda, ldb, ldc};
  const size_t room = ws_aligned ? workspace_bytes : 0;
  const int mode = !v.pointwise ? VIEW_GENERAL : (v.cstride > 1 && v.bsrc == B_NC ? VIEW_PREPASS : VIEW_DEFAULT);
  if (!s) {
    gensor_status st = memoised_schedule(p, vec_ok, mode, room, &local);
    if (st != GENSOR_OK) return st;
    s = &local;
  }
  const InstanceDesc* d = find_instance(s, v);
  if (d && !d->vec && (v.bsrc == B_KC || v.bsrc == B_NC) && !offsets_fit(*d, v, ld)) {
    // Rows too far apart for this tile's offsets (a schedule does not know the leading dimensions): the 64x64 tile of 16x16 blocks of
    // the instances at any alignment takes about twice as long ones.
    for (int i = 0; i < g_num_instances; ++i) {
      const InstanceDesc& e = g_instances[i];
      if (e.vec || e.mb != 16 || e.bm != 64 || !instance_serves(e, v) || !offsets_fit(e, v, ld)) continue;
      const int32_t panel = s->wg_remap, units = s->round_units;
      schedule_from_instance(e, &local);
      local.wg_remap = panel;
      local.round_units = units;
      s = &local;
      d = &e;
      break;
    }
  }
  if (!d) return GENSOR_ERR_NO_SCHEDULE;
  if (d->vec && !vec_ok) return GENSOR_ERR_NO_SCHEDULE;          // schedule asks for vector accesses the operands cannot give
  if (d->direct && !d->any_k() && v.bsrc != B_CONV && v.K % d->bk != 0) return GENSOR_ERR_NO_SCHEDULE;
  if (s->split_k < 1 || !split_allowed(*d, v, s->split_k)) return GENSOR_ERR_NO_SCHEDULE;
  SplitPlan sp = split_plan(*d, v, s->split_k, s->round_units);
  if (sp.split > 1 && room < sp.bytes) return GENSOR_ERR_WORKSPACE;
  if (!offsets_fit(*d, v, ld)) {
    // The same for aligned operands: what would be constructed of the tiles that reach, for the room there is.  (256-row tiles reach
    // half as far as 128-row ones, and which of them a shape gets is the cost model's choice: rows that ran must not depend on it.)
    const int32_t panel = s->wg_remap;
    const LeadingDims far = {same_reach(lda, v.esize, v.asrc == A_MC ? 256 : 0), same_reach(ldb, v.esize, v.bsrc == B_KC ? 0 : 256), same_reach(ldc, v.osize, 0)};
    if (!d->vec || memoised_schedule(p, vec_ok, mode, room, &local, &far) != GENSOR_OK) return GENSOR_ERR_UNSUPPORTED;
    d = find_instance(&local, v);
    if (!d) return GENSOR_ERR_UNSUPPORTED;
    local.wg_remap = panel;
    s = &local;
    sp = split_plan(*d, v, s->split_k, s->round_units);
  }

  KernelArgs a;
  std::memset(&a, 0, sizeof(a));
  a.A = A; a.B = B; a.C = C;
  a.M = (int32_t)v.M; a.N = (int32_t)v.N; a.K = (int32_t)v.K;
  a.lda = lda; a.ldb = ldb; a.ldc = ldc;
  a.strideA = strideA; a.strideB = strideB; a.strideC = strideC;
  a.alpha = alpha; a.beta = beta;
  // Write-through stores, except where rows of C that do not start on 128-byte lines make a large output: its partial lines
  // then go to memory one by one, where a write-back L2 joins them (outputs changing from call to call: 8192 x 8200 x 128
  // fp32 153 -> 70 us, 32 x 1000 x 1000 x 64 fp32 61 -> 36, with fp16 output 24.4 -> 20.4, 8192 x 3000 x 768 77.5 -> 66.8).
  // Smaller ones stay with write-through (6000 x 2500 fp32, 60 MB: 33.0 against 34.8 us; 4000 x 1000: 10.8 against
  // 11.8; 16-bit outputs of 8-30 MB: within 4 % either way), aligned rows too (48 x 768 x 768 x 64: 21.7 against 27.4).
  const int64_t c_bytes = v.batch * v.M * v.N * v.osize;
  const bool partial_lines = (ldc * v.osize) % 128 != 0 && c_bytes > (v.osize == 2 ? 32ll : 64ll) * 1024 * 1024;
  // Beside beta the line has just been read, and only large fp32 outputs (or launches of a single k tile, which wait on
  // little else) still gain from write-through.  With it and without, beta = 0.5: 96 x 1024 x 1024 x 64 269 against 277 us,
  // 8 of them 14.7 against 15.9, 4096^3 224.6 against 227.7, 6144 x 4096 x 512 126.4 against 128.0; but 4096 x 3072 x 768
  // 47.3 against 45.6, 4000 x 1000 x 512 21.9 against 17.7, and with 16-bit output 8192 x 3072 x 768 97.7 against 83.8,
  // 96 x 1024 x 1024 x 64 255 against 233, 16384 x 8192 x 512 554 against 532.
  const bool beside_beta = v.osize == 4 && (c_bytes >= 64ll * 1024 * 1024 || v.K <= d->bk);
  a.through = !partial_lines && (beta == 0.f || beside_beta);
  a.paired = v.osize == 2 && beta == 0.f && v.N % 2 == 0 && ldc % 2 == 0 && strideC % 2 == 0 && (reinterpret_cast<uintptr_t>(C) & 3u) == 0;
  a.tiles_m = (int32_t)((v.M + d->bm - 1) / d->bm);
  a.narrow = d->alternate() && sp.split == 1 && narrow_tiles(v, s->round_units > 0 ? s->round_units : gensor_hw_mi355x()->compute_units);
  const int bn = a.narrow ? 192 : d->bn;
  a.tiles_n = (int32_t)((v.N + bn - 1) / bn);
  a.batch = (int32_t)v.batch;
  a.panel = s->wg_remap > 0 ? s->wg_remap : 1;
  if (a.panel > a.tiles_m) a.panel = a.tiles_m;
  if ((int64_t)a.tiles_m * a.tiles_n * a.batch > INT32_MAX) return GENSOR_ERR_UNSUPPORTED;
  a.split = sp.split;
  a.whole = sp.split == 1 ? a.tiles_m * a.tiles_n * a.batch : (int32_t)sp.whole;
  // Read ahead where the launch moves more than the 256 MiB Infinity Cache holds (its operands then come from memory; from
  // that cache they come soon enough, and the wait at the end of each wave costs 2-10 %: 96 x 1024 x 1024 x 64 with fp16
  // output 61 -> 69 us, 48 x 768 x 768 x 64 21.1 -> 23.4), a batch is one or two k tiles deep, every XCD works through as many tiles (their count is
  // a multiple of 8; its range of them is contiguous) and the batch's workgroups cover the operands of the next with one
  // vector a thread; only the tiles such launches end in are compiled for it (Cfg::HAS_AHEAD); dense matrices only, so that every byte of the range is an element.
  if (v.batch > 1 && v.K <= 2 * d->bk && d->vec && sp.split == 1 && (v.bsrc == B_KC || v.bsrc == B_NC)) {
    const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
    const int64_t wa = strideA && lda == (v.asrc == A_KC ? v.K : v.M) ? v.M * v.K * v.esize : 0;
    const int64_t wb = strideB && ldb == (v.bsrc == B_KC ? v.K : v.N) ? v.N * v.K * v.esize : 0;
    const int64_t moved = v.batch * (wa + wb + v.M * v.N * v.osize);
    if (tiles * v.batch % 8 == 0 && moved > (int64_t)256 * 1024 * 1024 && wa + wb <= tiles * d->threads * 16) { a.ahead_a = wa; a.ahead_b = wb; }
  }
  // A launch of fewer k tiles than its instance has LDS stages touches that many stages only; allocating no more lets another workgroup
  // onto each compute unit, whose loads run under the others' stores.  fp32 output, us: 48 x 1024 x 1024 x 64 48.3 -> 40.6, 96 x 512 x 512
  // x 64 27.1 -> 24.3, 64 x 384 x 384 x 64 9.3 -> 8.3, 50 x 1000 x 1000 x 64 52.0 -> 46.2; 16-bit 64 x 384 x 384 x 64 7.3 -> 6.4, 50 x 1000 x 1000
  // x 64 41.1 -> 37.0.  Larger outputs lose to more of them storing at once.  Written through: fp32 8192 x 8192 x 64 45.4 -> 48.0, 7680 x 8192 x 64
  // 41.3 -> 44.5 (up to 210 MB a step that reads the output gains what the product loses, 50 x 1024 x 1024 x 64 34.4 -> 36.5, with a reader
  // 119.6 -> 114.9); 16-bit 48 x 1024 x 1024 x 64 (100 MB) with a reader 59.6 -> 66.0, 40 of them 50.1 -> 55.4, but 34 (71 MB) 41.3 -> 37.4.
  // Written back: fp32 8192 x 8200 x 64 (269 MB) 60.1 -> 63.7, 16384 x 5000 x 64 71.6 -> 77.5, but 60 x 1000 x 1000 x 64 63.7 -> 55.2; 16-bit at
  // every size (16384 x 8200 x 64 70.7 -> 67.3, 200 x 1000 x 1000 x 64 166 -> 132).  Where the next batch is read ahead, the stages it
  // does without are no gain, and with written back outputs a loss: 96 x 1024 x 1024 x 64 62.4 and 62.8, 64 x 1024 x 1152 x 64 49.0 and 54.2,
  // 96 x 1000 x 1000 x 64 85.4 and 102.9, 70 x 1020 x 1020 x 64 71.9 and 84.4.
  const bool ahead_form = d->vec && d->direct && d->stages == 2 && v.esize == 2 && v.osize == 4 && d->bm == 128 && d->bn == 128 && d->threads == 512;      // Cfg::HAS_AHEAD
  const bool ahead = ahead_form && a.ahead_a + a.ahead_b > 0;
  const int64_t most = v.osize == 2 ? (a.through ? 64ll * 1024 * 1024 : INT64_MAX) : (a.through ? 224ll : 256ll) * 1024 * 1024;
  const bool resident = !ahead && c_bytes <= most;
  const int64_t k_tiles = (v.K + d->bk - 1) / d->bk;
  a.lds_stages = resident && k_tiles < d->stages ? (int32_t)k_tiles : d->stages;
  a.partials = (float*)workspace;
  if (d->units) {
    ConvPlan pl;
    if (!conv_patch_plan(*d, v, &pl, s->round_units)) return GENSOR_ERR_NO_SCHEDULE;
    a.cTilePx = pl.tile_px;
    a.tiles_n = (int32_t)((v.N + pl.tile_px - 1) / pl.tile_px);
    if ((int64_t)a.tiles_m * a.tiles_n > INT32_MAX) return GENSOR_ERR_UNSUPPORTED;
    a.cN = (int32_t)p->n; a.cApitch = pl.a_pitch; a.cPatchRows = pl.patch_rows; a.cStageBytes = pl.stage_bytes;
    a.cInBytes = pl.in_bytes; a.cWBytes = pl.w_bytes; a.cOutBytes = pl.out_bytes;
    a.batch = 1;
  }
  if (d->conv_rows()) {
    ConvRowsPlan pl;
    if (!conv_rows_plan(d->bm, d->bn, v, &pl, s->round_units)) return GENSOR_ERR_NO_SCHEDULE;
    a.cTilePx = pl.tile_px;
    a.tiles_n = (int32_t)((v.N + pl.tile_px - 1) / pl.tile_px);
    if ((int64_t)a.tiles_m * a.tiles_n > INT32_MAX) return GENSOR_ERR_UNSUPPORTED;
    a.cN = (int32_t)p->n; a.cApitch = pl.a_pitch; a.cPatchRows = pl.rows; a.cStageBytes = pl.stage_bytes;
    a.cRowPitch = pl.row_pitch; a.cStageCh = pl.channels;
    const int64_t epc = 16 / v.esize, sc = (v.cs + epc - 1) / epc;
    const int64_t divisors[7] = {(pl.channels * v.cr * sc + 1) / 2 * 2, sc, (v.cw + epc - 1) / epc, pl.rows, v.ch + 2 * v.cpad, v.Q, v.P};
    for (int i = 0; i < 7; ++i) a.cRec[i] = divisors[i] > 1 ? (uint32_t)(((1ll << 32) + divisors[i] - 1) / divisors[i]) : 0u;
    a.cInBytes = pl.in_bytes; a.cWBytes = pl.w_bytes; a.cOutBytes = pl.out_bytes;
    a.batch = 1;
  }
  if (v.bsrc == B_CONV || v.bsrc == B_NCS2) {
    a.cC = (int32_t)p->c; a.cH = (int32_t)p->h; a.cW = (int32_t)p->w; a.cR = (int32_t)p->r; a.cS = (int32_t)p->s;
    a.cP = (int32_t)v.P; a.cQ = (int32_t)v.Q; a.cStride = (int32_t)p->stride; a.cPad = (int32_t)p->pad;
  }
  hipError_t e = sp.split > 1 ? d->launch_split(a, (hipStream_t)stream) : d->launch(a, (hipStream_t)stream);
  if (e == hipSuccess && sp.split > 1) e = launch_split_reduce(*d, a, (hipStream_t)stream);
  return e == hipSuccess ? GENSOR_OK : GENSOR_ERR_DEVICE;
}
}  // namespace

extern "C" gensor_status gensor_bmm(const gensor_schedule* s, const gensor_problem* p, float alpha,
                                    const void* A, int64_t lda, int64_t strideA,
                                    const void* B, int64_t ldb, int64_t strideB,
                                    float beta, void* C, int64_t ldc, int64_t strideC,
                                    void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p || !A || !B || !C) return GENSOR_ERR_INVALID_ARG;
  if (p->op != GENSOR_OP_GEMM && p->op != GENSOR_OP_BMM) return GENSOR_ERR_INVALID_ARG;
  GemmView v;
  gensor_status st = gemm_view(p, &v);
  if (st != GENSOR_OK) return st;
  if (lda < (v.asrc == A_KC ? v.K : v.M)) return GENSOR_ERR_INVALID_ARG;
  if (ldb < (v.bsrc == B_KC ? v.K : v.N)) return GENSOR_ERR_INVALID_ARG;
  if (ldc < v.N) return GENSOR_ERR_INVALID_ARG;
  if (strideA < 0 || strideB < 0 || strideC < 0) return GENSOR_ERR_INVALID_ARG;
  if (v.batch > 1 && strideC < v.M * ldc - (ldc - v.N)) return GENSOR_ERR_INVALID_ARG;   // outputs must not overlap
  return run(s, p, v, alpha, A, lda, strideA, B, ldb, strideB, beta, C, ldc, strideC, workspace, workspace_bytes, hip_stream);
}

extern "C" gensor_status gensor_gemm(const gensor_schedule* s, const gensor_problem* p, float alpha,
                                     const void* A, int64_t lda, const void* B, int64_t ldb,
                                     float beta, void* C, int64_t ldc,
                                     void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p || p->op != GENSOR_OP_GEMM) return GENSOR_ERR_INVALID_ARG;
  return gensor_bmm(s, p, alpha, A, lda, 0, B, ldb, 0, beta, C, ldc, 0, workspace, workspace_bytes, hip_stream);
}

// ------------------------------------------------------------------------------------
// gensor_gemm for callers that cannot bring a workspace: the split-k partial tiles live in a device array that is part of this library's code object.
// ------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[GENSOR_STATIC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mutex;
void* g_scratch_ptr[64];          // per device ordinal: where that device's copy of `scratch` lives

// The address of this device's copy of the array (each device holds its own, at its own address);
// looked up once per device, with that device current.
gensor_status static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return GENSOR_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return GENSOR_ERR_DEVICE;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return GENSOR_OK;
}
}  // namespace

extern "C" gensor_status gensor_gemm_static_scratch(const gensor_schedule* s, const gensor_problem* p, float alpha,
                                                    const void* A, int64_t lda, const void* B, int64_t ldb,
                                                    float beta, void* C, int64_t ldc, void* hip_stream) {
  if (!p || p->op != GENSOR_OP_GEMM) return GENSOR_ERR_INVALID_ARG;
  if (s && gensor_workspace_bytes(s, p) > (size_t)GENSOR_STATIC_SCRATCH_BYTES) return GENSOR_ERR_WORKSPACE;
  void* ptr = nullptr;
  gensor_status st = static_scratch(&ptr);
  if (st != GENSOR_OK) return st;
  // from here on the array is a workspace like any other: the partial tiles are written before they are read
  return gensor_bmm(s, p, alpha, A, lda, 0, B, ldb, 0, beta, C, ldc, 0, ptr, (size_t)GENSOR_STATIC_SCRATCH_BYTES, hip_stream);
}

extern "C" gensor_status gensor_conv2d(const gensor_schedule* s, const gensor_problem* p,
                                       const void* input, const void* weight, void* output,
                                       void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p || !input || !weight || !output || p->op != GENSOR_OP_CONV2D) return GENSOR_ERR_INVALID_ARG;
  GemmView v;
  gensor_status st = gemm_view(p, &v);
  if (st != GENSOR_OK) return st;
  if (v.pointwise) {
    // one GEMM per image: A = filters [k][c] shared by all images, B = the (sampled) input
    // [c][P*Q] of the image, C = its output [k][P*Q].  Views are tried in order of
    // preference: sampled while fetched (stride 2, no workspace), compacted by a pre-pass
    // (needs the workspace), then the general implicit GEMM.  An explicit schedule selects
    // the view whose instance it names.
    const int64_t PQ = v.N;
    for (int mode = VIEW_DEFAULT; mode <= VIEW_PREPASS; ++mode) {
      GemmView w;
      st = gemm_view(p, &w, mode);
      if (st != GENSOR_OK) return st;
      if (mode == VIEW_PREPASS && w.bsrc == v.bsrc) break;          // the same view again
      const size_t need = pointwise_workspace(w);
      const bool have = need == 0 || (workspace && (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0 && workspace_bytes >= need);
      const int64_t ldb = need ? PQ : p->h * p->w;
      if (s) {
        if (!find_instance(s, w)) continue;
        if (!have) return GENSOR_ERR_WORKSPACE;
      } else {
        if (!have) continue;
        if (w.bsrc == B_NCS2 && !vector_ok(w, weight, w.K, 0, input, ldb, w.K * ldb)) continue;   // sampled instances are vector-only
      }
      const void* X = input;
      if (need) {
        const int64_t planes = p->n * p->c;
        const int epc = 16 / w.esize;
        const int64_t threads = (planes * PQ + epc - 1) / epc;
        if ((threads + 255) / 256 > INT32_MAX) return GENSOR_ERR_UNSUPPORTED;
        const unsigned blocks = (unsigned)((threads + 255) / 256);
        if (w.esize == 4)
          hipLaunchKernelGGL(subsample_input<4>, dim3(blocks), dim3(256), 0, (hipStream_t)hip_stream, input, workspace, planes,
                             (int)p->h, (int)p->w, (int)w.P, (int)w.Q, (int)p->stride);
        else
          hipLaunchKernelGGL(subsample_input<2>, dim3(blocks), dim3(256), 0, (hipStream_t)hip_stream, input, workspace, planes,
                             (int)p->h, (int)p->w, (int)w.P, (int)w.Q, (int)p->stride);
        if (hipGetLastError() != hipSuccess) return GENSOR_ERR_DEVICE;
        X = workspace;
      }
      return run(s, p, w, 1.0f, weight, w.K, 0, X, ldb, w.K * ldb, 0.0f, output, PQ, w.M * PQ, nullptr, 0, hip_stream);
    }
    st = gemm_view(p, &v, VIEW_GENERAL);
    if (st != GENSOR_OK) return st;
  }
  // A = filters [k][c*r*s] (k-contiguous), B = gathered input, C = output viewed per image.
  return run(s, p, v, 1.0f, weight, v.K, 0, input, 0, 0, 0.0f, output, v.N, 0, workspace, workspace_bytes, hip_stream);
}
