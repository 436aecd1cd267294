// The two memory-bound operators of the paper's benchmark: GEMV and AvgPooling2d (operator
// table, GEMV and AvgPooling2d rows).  Neither is a contraction worth a matrix core: both
// stream their input once from HBM, so the kernels are plain coalesced vector loads, fp32
// arithmetic on the vector ALUs and one store per output.
#include <hip/hip_runtime.h>

#include "../../include/gensor.h"
#include "gemm_kernel.hpp"

namespace gensor {

// 16 bytes of stored elements -> fp32 values
template <typename T>
__device__ inline void unpack_chunk(const u32x4& v, float* f) {
  if constexpr (ElemSize<T>::value == 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = as_f32(v[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint16_t bits = (uint16_t)(v[e >> 1] >> ((e & 1) * 16));
      f[e] = to_float<T>(&bits, 0);
    }
  }
}

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// ---------------------------------------------------------------------------------------
// GEMV, y_i = alpha * sum_n A_in x_n + beta * y_i.  Bound by reading A once: what it needs is enough bytes in flight on
// every CU and no wait that another load does not cover.  A wave takes ROWS rows (every x vector it reads serves all of
// them) and UNROLL 16-byte vectors of each per trip, all requested together with the x vectors; x comes through the L1
// (it is used by every wave of the CU) rather than through LDS panels, whose fill and barrier stood in front of the
// first product.  SPLIT waves share their rows, taking turns at the vectors: a trip then covers SPLIT times as much of
// a row, and few rows still occupy the chip.  Rows may start anywhere: a 16-byte load takes any address (element
// loads, used before for rows off the 16-byte boundaries, reached 2 TB/s).  The vectors counted here lie wholly inside
// a row; what is left of it is read element by element.
// Same-run A/B against 32 KB panels of x, fp16, inputs changing from call to call: 16384 x 16384 91.7 -> 75.7 us (7.1
// TB/s), 16384 x 8192 51.5 -> 40.2, 16384 x 8191 128 -> 44, 4096 x 8192 12.9 -> 11.2, 1024 x 5003 25.4 -> 3.9,
// 16384 x 1000 8.8 -> 6.6.
// ---------------------------------------------------------------------------------------
typedef u32x4 __attribute__((aligned(2))) u32x4_any;       // 16 bytes at any element's address

// STREAM: the rows of A are read with the non-temporal hint.  A matrix that does not fit the 256 MiB Infinity Cache
// together with x and y only evicts itself from it (16384 x 16384 fp16: 81.4 -> 75.7 us with the hint, 16384 x 8192:
// 43.6 -> 40.2); one that fits is served from it on repeated calls and loses that (4096 x 8192: 11.2 -> 12.4).
template <bool STREAM>
__device__ inline u32x4 load_row_vector(const char* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load((const u32x4_any*)p);
  else return *(const u32x4_any*)p;
}

template <typename T, bool STREAM, int SPLIT>
__global__ __launch_bounds__(256) void gemv_kernel(const char* A, int64_t lda, const char* x, float* y, int M, int N, float alpha,
                                                   float beta) {
  constexpr int ES = ElemSize<T>::value, EPC = 16 / ES, ROWS = 2, UNROLL = 4;
  __shared__ float part_sums[4][ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, part = wave % SPLIT;
  const int row0 = (int)((blockIdx.x * (4 / SPLIT) + wave / SPLIT) * ROWS);
  const char* a[ROWS];
  float acc[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    a[r] = A + (int64_t)(row0 + r < M ? row0 + r : 0) * lda * ES;
    acc[r] = 0.f;
  }
  const int full = N / EPC, rem = N - full * EPC;          // whole vectors of a row, elements behind them
  for (int c = part * 64 + lane; c < full; c += 64 * SPLIT * UNROLL) {
    u32x4 xv[UNROLL], av[UNROLL][ROWS];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int64_t off = (int64_t)(c + u * 64 * SPLIT) * 16;
      xv[u] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int r = 0; r < ROWS; ++r) av[u][r] = u32x4{0u, 0u, 0u, 0u};
      if (c + u * 64 * SPLIT < full) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) av[u][r] = load_row_vector<STREAM>(a[r] + off);
        xv[u] = *(const u32x4_any*)(x + off);
      }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      float fx[EPC];
      unpack_chunk<T>(xv[u], fx);
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        float fa[EPC];
        unpack_chunk<T>(av[u][r], fa);
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[r] = fmaf(fa[e], fx[e], acc[r]);
      }
    }
  }
  if (part == 0 && lane < rem) {                           // lane e takes element e of the partial vector
    const int64_t i = (int64_t)full * EPC + lane;
    const float xl = to_float<T>(x, i);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = fmaf(to_float<T>(a[r], i), xl, acc[r]);
  }
#pragma unroll
  for (int r = 0; r < ROWS; ++r) acc[r] = wave_sum(acc[r]);
  if constexpr (SPLIT > 1) {
    if (lane == 0)
#pragma unroll
      for (int r = 0; r < ROWS; ++r) part_sums[wave][r] = acc[r];
    __syncthreads();
    if (part) return;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      acc[r] = part_sums[wave][r];
#pragma unroll
      for (int p = 1; p < SPLIT; ++p) acc[r] += part_sums[wave + p][r];
    }
  }
  if (lane < ROWS && row0 + lane < M) {
    const float sum = lane ? acc[1] : acc[0];
    y[row0 + lane] = alpha * sum + (beta != 0.f ? beta * y[row0 + lane] : 0.f);
  }
}

// ---------------------------------------------------------------------------------------
// AvgPooling2d, O[plane][p][q] = (1/F^2) sum_{i,j<F} I[plane][S p + i][S q + j].  The window
// is summed in fp32 and divided once by F*F.
//
// avgpool_lds_kernel: the input a workgroup needs is one contiguous span of the NCHW tensor
// (whole planes, or the rows under a run of output rows of one plane).  It is brought into
// LDS with aligned 16-byte vector loads (2-byte loads per window element would make the load
// pipeline, not HBM, the limit), and the windows are then read from LDS.
// Bound by HBM.  Whole planes are read, and fp32 outputs stored, non-temporal where the input alone is more than the last cache keeps
// (STREAM): 128 x 168 x 83 x 83 fp16 83.5 -> 80.7 us (441 MB: 5.5 TB/s), fp32 135 -> 117.  Smaller inputs may still be there from the
// step that wrote them (32 x 168 x 83 x 83 fp16 21.1 -> 22.9 with the hint), and runs of rows read the rows between two of them twice.
// fp32 outputs that the L2s hold are stored non-temporal, too (THROUGH): they take no room from the input that neighbours share lines of, and the
// step that reads them finds no dirty lines in front of it (pooling alone, and with a reader behind it: 16 x 96 x 83 x 83 fp16, 10 MB, 9.7 -> 8.9,
// 16.4 -> 14.0; 32 x 64 x 112 x 112 fp16, 26 MB, 19.2 -> 17.7, 27.8 level; 16 x 64 x 112 x 112 fp32, 13 MB, 15.7 -> 14.8, 21.0 -> 20.6).  Beyond,
// pooling alone gains less than its reader loses (64 x 168 x 83 x 83 fp16, 72 MB, 38.3 level, 60.7 -> 63.9; 16 x 48 x 299 x 299 fp32, 68 MB,
// 65.5 -> 63.5, 85.0 -> 92.5; 16 x 168 x 83 x 83 fp32, 18 MB, 17.9 -> 17.8, 24.9 -> 25.8).
// avgpool_direct_kernel: one thread per output straight from global memory, for inputs that
// are not 16-byte aligned or whose rows do not fit the LDS span.
// ---------------------------------------------------------------------------------------
constexpr int POOL_SPAN_BYTES = 32768;
constexpr int POOL_VECS = (POOL_SPAN_BYTES + 16 + 15) / 16 / 256 + 1;     // 16-byte vectors per thread covering span + skew

template <typename T, typename OutT, bool STREAM, bool THROUGH>
__global__ __launch_bounds__(256) void avgpool_lds_kernel(const char* in, void* out, int64_t in_bytes, int planes, int H, int W, int P,
                                                          int Q, int F, int S, int planes_per_wg, int rows_per_wg, int chunks_per_plane) {
  constexpr int ES = ElemSize<T>::value;
  extern __shared__ __attribute__((aligned(16))) char span[];      // the launch sizes it to this problem's span (+ skew)
  const int tid = threadIdx.x;
  const int group = blockIdx.x / chunks_per_plane, chunk = blockIdx.x - group * chunks_per_plane;
  const int plane0 = group * planes_per_wg;
  const int nplanes = min(planes_per_wg, planes - plane0);
  const int p0 = chunk * rows_per_wg;
  const int nrows = min(rows_per_wg, P - p0);
  // span of input elements [e0, e0 + len)
  const int64_t e0 = ((int64_t)plane0 * H + (int64_t)S * p0) * W;
  const int len = chunks_per_plane == 1 ? nplanes * H * W : ((nrows - 1) * S + F) * W;
  const int64_t b0 = e0 * ES, a0 = b0 & ~(int64_t)15;
  const int skew = (int)(b0 - a0);                            // bytes before the first element in LDS
  const int nvec = (skew + len * ES + 15) / 16;
  // all of a thread's vectors are requested before the first one is written to LDS (one memory
  // round trip per workgroup instead of one per vector); the span holds at most POOL_VECS per thread
  u32x4 d[POOL_VECS];
#pragma unroll
  for (int i = 0; i < POOL_VECS; ++i) {
    const int v = tid + i * 256;
    const int64_t addr = a0 + (int64_t)v * 16;
    d[i] = u32x4{0u, 0u, 0u, 0u};
    if (v < nvec) {
      if (addr + 16 <= in_bytes) {
        if constexpr (STREAM) d[i] = __builtin_nontemporal_load((const u32x4*)(in + addr));
        else d[i] = *(const u32x4*)(in + addr);
      } else {                                                // last vector of the tensor: element by element
        for (int e = 0; e < 16 / ES; ++e) {
          if (addr + (e + 1) * ES <= in_bytes) {
            if constexpr (ES == 4) d[i][e] = *(const uint32_t*)(in + addr + e * 4);
            else d[i][e >> 1] |= (uint32_t)*(const uint16_t*)(in + addr + e * 2) << ((e & 1) * 16);
          }
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < POOL_VECS; ++i) {
    const int v = tid + i * 256;
    if (v < nvec) *(u32x4*)(span + v * 16) = d[i];
  }
  __syncthreads();
  const int per_plane = nrows * Q;
  const int total = nplanes * per_plane;
  const float count = (float)(F * F);
  // thread t takes outputs t, t + 256, ...; (plane, row, column) advance incrementally
  int g = tid / per_plane, pr, q;
  {
    const int r = tid - g * per_plane;
    pr = r / Q;
    q = r - pr * Q;
  }
  const int dq = 256 % Q, dp = 256 / Q;
  for (int t = tid; t < total; t += 256) {
    const int base = (g * H + S * pr) * W + S * q;            // element offset inside the span
    float acc = 0.f;
    for (int i = 0; i < F; ++i)
      for (int j = 0; j < F; ++j) acc += to_float<T>(span + skew, base + i * W + j);
    const int64_t o = ((int64_t)(plane0 + g) * P + p0 + pr) * Q + q;
    if constexpr (THROUGH) __builtin_nontemporal_store(acc / count, (float*)out + o);
    else store_out<OutT>(out, o, acc / count);
    q += dq;
    pr += dp;
    if (q >= Q) { q -= Q; ++pr; }
    while (pr >= nrows) { pr -= nrows; ++g; }
  }
}

template <typename T, typename OutT>
__global__ __launch_bounds__(256) void avgpool_direct_kernel(const void* in, void* out, int64_t total, int H, int W, int P, int Q, int F,
                                                             int S) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int64_t t = idx / Q;
  const int q = (int)(idx - t * Q);
  const int64_t plane = t / P;
  const int p = (int)(t - plane * P);
  const int64_t base = (plane * H + (int64_t)S * p) * W + (int64_t)S * q;
  float acc = 0.f;
  for (int i = 0; i < F; ++i)
    for (int j = 0; j < F; ++j) acc += to_float<T>(in, base + (int64_t)i * W + j);
  store_out<OutT>(out, idx, acc / (float)(F * F));
}

// Four waves share two rows where that leaves each a trip's worth of vectors (256 vectors a row: at 250 both splits take
// 10.7-10.9 us for 16384 rows, at 475 the shared rows 20.8 against 22.7 us, at 125 9.2 against 7.0), and where the launch
// can hold that many workgroups: HIP takes fewer than 2^32 threads, 2^25 rows at two a workgroup, four times that otherwise.
template <typename T>
hipError_t launch_gemv(const void* A, int64_t lda, const void* x, float* y, int64_t M, int64_t N, float alpha, float beta, hipStream_t st) {
  constexpr int ES = ElemSize<T>::value, EPC = 16 / ES;
  const bool stream = M * lda * ES + N * ES + M * 4 > (int64_t)256 * 1024 * 1024;
  const bool shared = N / EPC >= 256 && (M + 1) / 2 * 256 < ((int64_t)1 << 32);
  const dim3 grid((unsigned)(shared ? (M + 1) / 2 : (M + 7) / 8)), block(256);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, (const char*)A, lda, (const char*)x, y, (int)M, (int)N, alpha, beta); };
  if (shared) stream ? go(gemv_kernel<T, true, 4>) : go(gemv_kernel<T, false, 4>);
  else stream ? go(gemv_kernel<T, true, 1>) : go(gemv_kernel<T, false, 1>);
  return hipGetLastError();
}

template <typename T, typename OutT>
hipError_t launch_pool(const void* in, void* out, int64_t planes, int64_t h, int64_t w, int64_t f, int64_t s, hipStream_t st) {
  constexpr int ES = ElemSize<T>::value;
  const int64_t P = (h - f) / s + 1, Q = (w - f) / s + 1;
  const int64_t plane_bytes = h * w * ES, row_bytes = w * ES;
  const bool aligned = (reinterpret_cast<uintptr_t>(in) & 15u) == 0;
  int64_t G = 0, R = 0, cpp = 0;
  if (aligned && plane_bytes <= POOL_SPAN_BYTES) {             // whole planes per workgroup
    G = POOL_SPAN_BYTES / plane_bytes;
    const int64_t cap = (8192 + P * Q - 1) / (P * Q);          // keep a workgroup to a few thousand outputs
    if (G > cap) G = cap;
    // enough workgroups to keep every CU's resident set (LDS is sized to the span) turning over several times
    const int64_t spread = planes / (256 * 8 * 4);
    if (G > spread) G = spread > 1 ? spread : 1;
    if (G > planes) G = planes;
    R = P;
    cpp = 1;
  } else if (aligned && f * row_bytes <= POOL_SPAN_BYTES) {    // runs of output rows of one plane
    G = 1;
    R = (POOL_SPAN_BYTES / row_bytes - f) / s + 1;
    if (R > P) R = P;
    cpp = (P + R - 1) / R;
  }
  const int64_t groups = G ? (planes + G - 1) / G * cpp : 0;
  if (G && groups <= INT32_MAX && planes <= INT32_MAX) {
    const int64_t span_elems = cpp == 1 ? G * h * w : ((R - 1) * s + f) * w;
    const size_t lds_bytes = (size_t)((span_elems * ES + 15 + 15) / 16 * 16 + 16);      // span + skew, whole vectors
    constexpr bool FP32_OUT = ElemSize<OutT>::value == 4;
    const bool stream = cpp == 1 && planes * plane_bytes > 256ll * 1024 * 1024;
    const bool through = planes * P * Q * 4 <= (ES == 2 ? 32ll : 16ll) * 1024 * 1024;
    const auto kernel = stream ? avgpool_lds_kernel<T, OutT, true, FP32_OUT>
                               : through ? avgpool_lds_kernel<T, OutT, false, FP32_OUT> : avgpool_lds_kernel<T, OutT, false, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(256), lds_bytes, st, (const char*)in, out, planes * plane_bytes, (int)planes,
                       (int)h, (int)w, (int)P, (int)Q, (int)f, (int)s, (int)G, (int)R, (int)cpp);
  } else {
    const int64_t total = planes * P * Q;
    hipLaunchKernelGGL((avgpool_direct_kernel<T, OutT>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, in, out, total, (int)h,
                       (int)w, (int)P, (int)Q, (int)f, (int)s);
  }
  return hipGetLastError();
}

}  // namespace gensor

using namespace gensor;

extern "C" gensor_status gensor_gemv(gensor_dtype in_dtype, int64_t M, int64_t N, float alpha, const void* A, int64_t lda,
                                     const void* x, float beta, float* y, void* hip_stream) {
  if (!A || !x || !y || M <= 0 || N <= 0 || lda < N) return GENSOR_ERR_INVALID_ARG;
  // HIP takes fewer than 2^32 threads, 256 for eight rows; a trip past the end of a row, 64 * SPLIT * UNROLL vectors of at most
  // 8 elements, is counted in an int
  if (M > ((int64_t)1 << 27) - 8 || N > INT32_MAX - 32768) return GENSOR_ERR_UNSUPPORTED;
  hipError_t e;
  switch (in_dtype) {
    case GENSOR_F32: e = launch_gemv<f32_t>(A, lda, x, y, M, N, alpha, beta, (hipStream_t)hip_stream); break;
    case GENSOR_F16: e = launch_gemv<f16_t>(A, lda, x, y, M, N, alpha, beta, (hipStream_t)hip_stream); break;
    case GENSOR_BF16: e = launch_gemv<bf16_t>(A, lda, x, y, M, N, alpha, beta, (hipStream_t)hip_stream); break;
    default: return GENSOR_ERR_INVALID_ARG;
  }
  return e == hipSuccess ? GENSOR_OK : GENSOR_ERR_DEVICE;
}

extern "C" gensor_status gensor_avgpool2d(gensor_dtype in_dtype, gensor_dtype out_dtype, int64_t n, int64_t c, int64_t h, int64_t w,
                                          int64_t f, int64_t stride, const void* input, void* output, void* hip_stream) {
  if (!input || !output || n <= 0 || c <= 0 || h <= 0 || w <= 0 || f <= 0 || stride <= 0 || f > h || f > w) return GENSOR_ERR_INVALID_ARG;
  if (in_dtype != GENSOR_F32 && in_dtype != GENSOR_F16 && in_dtype != GENSOR_BF16) return GENSOR_ERR_INVALID_ARG;
  if (out_dtype != GENSOR_F32 && out_dtype != in_dtype) return GENSOR_ERR_UNSUPPORTED;
  const int64_t P = (h - f) / stride + 1, Q = (w - f) / stride + 1;
  if (h > INT32_MAX || w > INT32_MAX || f > 4096 || (n * c * P * Q + 255) / 256 > INT32_MAX) return GENSOR_ERR_UNSUPPORTED;
  hipStream_t st = (hipStream_t)hip_stream;
  const int64_t planes = n * c;
  hipError_t e;
  if (in_dtype == GENSOR_F32) e = launch_pool<f32_t, f32_t>(input, output, planes, h, w, f, stride, st);
  else if (in_dtype == GENSOR_F16)
    e = out_dtype == GENSOR_F32 ? launch_pool<f16_t, f32_t>(input, output, planes, h, w, f, stride, st)
                                : launch_pool<f16_t, f16_t>(input, output, planes, h, w, f, stride, st);
  else
    e = out_dtype == GENSOR_F32 ? launch_pool<bf16_t, f32_t>(input, output, planes, h, w, f, stride, st)
                                : launch_pool<bf16_t, bf16_t>(input, output, planes, h, w, f, stride, st);
  return e == hipSuccess ? GENSOR_OK : GENSOR_ERR_DEVICE;
}
