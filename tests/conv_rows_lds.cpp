// Where the row-staged convolution's lanes read and write LDS, walked on the host with the kernel's own window arithmetic: every
// access of every lane and step has to lie inside the workgroup's allocation.  Run by tests/test_conv_rows_lds.py.
#include <cstdio>
#include <cstring>

#include "conv_rows_kernel.hpp"
#include "host_common.hpp"

using namespace gensor;

static int failures = 0, walked = 0;

template <bool ONE_CHUNK>
static int64_t furthest_read(const GemmView& v, const ConvRowsPlan& pl, int64_t n0, int channels) {
  const int epc = 16 / v.esize, sc = (int)((v.cs + epc - 1) / epc), xo = (int)((v.cpad + epc - 1) / epc) * epc;
  const int64_t hp = v.ch + 2 * v.cpad;
  const int chan_pitch = pl.rows * pl.row_pitch, nch = channels * (int)v.cr * sc, steps = (nch + 1) / 2;
  const int64_t g0 = n0 / v.Q, r0 = (g0 / v.P) * hp + (g0 % v.P) * v.cstride;
  uint32_t reach = 0;                                          // of all chunks and both lane groups, relative to a window
  for (int group = 0; group < 2; ++group) {
    RowsWalk<ONE_CHUNK> walk;
    if (group) walk.advance((int)v.cr, sc, pl.row_pitch, chan_pitch);
    const uint32_t last = walk.last(channels, (int)v.cr, sc, pl.row_pitch, chan_pitch);
    for (int s = 0; s < steps; ++s) {
      if (2 * s + group < nch && walk.at(last) != walk.off) { std::printf("chunk %d of %d moved\n", 2 * s + group, nch); ++failures; }
      if (walk.at(last) > reach) reach = walk.at(last);
      walk.advance((int)v.cr, sc, pl.row_pitch, chan_pitch);
      walk.advance((int)v.cr, sc, pl.row_pitch, chan_pitch);
    }
  }
  const int64_t N = v.cn * v.P * v.Q, n1 = n0 + pl.tile_px < N ? n0 + pl.tile_px : N;
  int64_t far = 0;
  for (int64_t n = n0; n < n1; ++n) {
    const int64_t g = n / v.Q, img = g / v.P, p = g % v.P, q = n % v.Q;
    const uint32_t at = rows_window((int)(img * hp + p * v.cstride - r0), (int)(q * v.cstride - v.cpad + xo), pl.row_pitch, v.esize);
    const int64_t end = (int64_t)(at & ~3u) + reach + (v.esize == 2 ? 20 : 16);
    if (end > far) far = end;
  }
  return far;
}

static void check(int dtype, int64_t n, int64_t c, int64_t h, int64_t w, int64_t k, int64_t r, int64_t s, int64_t stride, int64_t pad) {
  gensor_problem p;
  std::memset(&p, 0, sizeof(p));
  p.op = GENSOR_OP_CONV2D; p.in_dtype = dtype; p.out_dtype = GENSOR_F32;
  p.n = n; p.c = c; p.h = h; p.w = w; p.k = k; p.r = r; p.s = s; p.stride = stride; p.pad = pad;
  GemmView v;
  if (gemm_view(&p, &v, VIEW_GENERAL) != GENSOR_OK) { std::printf("no view\n"); ++failures; return; }
  for (int i = 0; i < g_num_instances; ++i) {
    const InstanceDesc& d = g_instances[i];
    ConvRowsPlan pl;
    if (!d.conv_rows() || !instance_serves(d, v) || !conv_rows_plan(d.bm, d.bn, v, &pl)) continue;
    ++walked;
    const int epc = 16 / v.esize;
    const int64_t input_bytes = pl.stage_bytes - (int64_t)d.bm * pl.a_pitch, N = v.cn * v.P * v.Q;
    const int64_t nche = (pl.channels * v.cr * ((v.cs + epc - 1) / epc) + 1) / 2 * 2;
    const int64_t xo = (v.cpad + epc - 1) / epc * epc, segs = (v.cw + epc - 1) / epc;
    if (nche * 16 > pl.a_pitch) { std::printf("filter row %lld over pitch %d\n", (long long)nche * 16, pl.a_pitch); ++failures; }
    const int64_t written = ((int64_t)pl.channels * pl.rows - 1) * pl.row_pitch + (xo + segs * epc) * v.esize;
    if (written > input_bytes || pl.stage_bytes > 160 * 1024) { std::printf("stage of %d bytes\n", pl.stage_bytes); ++failures; }
    // the rows a tile can touch, counted over every row it may start at
    const int64_t hp = v.ch + 2 * v.cpad, last_row = v.cn * v.P - 1;
    int64_t out_rows = pl.tile_px % v.Q == 0 ? pl.tile_px / v.Q : (pl.tile_px + v.Q - 2) / v.Q + 1, rows = 0;
    if (out_rows > last_row + 1) out_rows = last_row + 1;
    for (int64_t first = 0; first < v.P; ++first) {
      const int64_t g = first + out_rows - 1 < last_row ? first + out_rows - 1 : last_row;
      const int64_t r = (g / v.P) * hp + (g % v.P - first) * v.cstride + v.cr;
      if (r > rows) rows = r;
    }
    if (rows != pl.rows) { std::printf("%d rows planned, %lld touched\n", pl.rows, (long long)rows); ++failures; }
    const int tail = (int)(v.cc % pl.channels ? v.cc % pl.channels : pl.channels);       // channels of the last stage
    for (int64_t n0 = 0; n0 < N; n0 += pl.tile_px) {
      for (int ch : {pl.channels, tail}) {
        const int64_t far = v.cs <= epc ? furthest_read<true>(v, pl, n0, ch) : furthest_read<false>(v, pl, n0, ch);
        if (far > input_bytes) {
          std::printf("dtype %d %lldx%lldx%lldx%lld %lldx%lld tile %dx%d at pixel %lld: reads %lld of %lld bytes\n", dtype, (long long)n, (long long)c,
                      (long long)h, (long long)w, (long long)r, (long long)s, d.bm, d.bn, (long long)n0, (long long)far, (long long)input_bytes);
          ++failures;
          return;
        }
      }
    }
  }
}

int main() {
  for (int dt : {GENSOR_F16, GENSOR_BF16, GENSOR_F32}) {
    check(dt, 16, 3, 112, 112, 64, 7, 7, 2, 3);      // an odd number of chunks per stage
    check(dt, 3, 3, 33, 31, 70, 7, 7, 2, 3);
    check(dt, 1, 1, 9, 300, 5, 5, 5, 1, 2);
    check(dt, 2, 7, 13, 12, 33, 3, 3, 1, 1);
    check(dt, 2, 5, 11, 17, 32, 1, 1, 3, 1);
    check(dt, 1, 4, 20, 21, 16, 2, 9, 1, 4);         // a filter row of several chunks
    check(dt, 1, 2, 40, 40, 8, 17, 17, 2, 0);
    check(dt, 4, 40, 6, 6, 64, 5, 5, 1, 2);          // several stages, the last one partial
    check(dt, 1, 3, 8, 8, 130, 3, 3, 1, 5);
    check(dt, 16, 16, 112, 112, 64, 5, 5, 1, 2);
    check(dt, 2, 6, 50, 61, 48, 7, 7, 1, 3);
    check(dt, 1, 1, 1, 1, 1, 1, 1, 1, 0);
    check(dt, 5, 1, 4, 3, 9, 3, 3, 3, 1);            // several images to a tile, strides beyond the filter
    check(dt, 2, 1, 4, 3, 9, 2, 2, 2, 0);
    check(dt, 30, 2, 11, 5, 33, 4, 2, 3, 2);
    check(dt, 1, 2, 700, 1, 8, 5, 1, 1, 2);          // one column
  }
  std::printf("%s: %d plans, %d failure(s)\n", failures ? "FAILED" : "inside", walked, failures);
  return failures || walked < 100 ? 1 : 0;
}
