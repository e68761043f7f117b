// Row-wise pieces of the decoder layer around the DAF attention, on the rows
// the layer recomputes (the important and question rows: Sec. 2 item 2, the
// QKV computation phase; Sec. 2 item 3, the compact fused state feeds the next
// layer): RMSNorm before the projections, the rotary position embedding of
// q and k at each row's original position, and the MLP gate SiLU(g) * u.
// All HBM-bound; bf16 in and out, fp32 arithmetic (the rotation angle in
// fp64, since positions reach 10^5).
#include "daf_internal.h"

namespace daf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kRowThreads = 256;  // 4 waves, one row each

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// y = x / sqrt(mean(x^2) + eps) * w, one wave per row, 16-byte pieces.
__global__ __launch_bounds__(kRowThreads) void rmsnorm_kernel(int64_t rows, int width, const __bf16 *x,
                                                              const __bf16 *w, float eps, __bf16 *y) {
  const int64_t row = (int64_t)blockIdx.x * (kRowThreads / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63;
  const int pieces = width / 8;
  const bf16x8 *xr = reinterpret_cast<const bf16x8 *>(x + row * width);
  float ss = 0.f;
  for (int j = lane; j < pieces; j += 64) {
    const bf16x8 v = xr[j];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float f = (float)v[e];
      ss = __builtin_fmaf(f, f, ss);
    }
  }
  const float inv = 1.0f / sqrtf(wave_sum(ss) / (float)width + eps);
  const bf16x8 *wr = reinterpret_cast<const bf16x8 *>(w);
  bf16x8 *yr = reinterpret_cast<bf16x8 *>(y + row * width);
  for (int j = lane; j < pieces; j += 64) {
    const bf16x8 v = xr[j], g = wr[j];
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (__bf16)((float)v[e] * inv * (float)g[e]);
    yr[j] = o;
  }
}

// In place: features (i, i + D/2) of every head rotate by pos * theta^(-2i/D).
//
// A workgroup takes kRopeRows rows of up to two tensors (q and k of a layer in
// one launch). The angle depends on neither the head nor the tensor: each
// thread computes the sine and cosine of one (row, i) in fp64 into LDS, then
// the threads go over the rows' heads in 16-byte pieces of each half. HBM-bound
// (every value read and written once). It replaces a thread per (row, i) that
// went through the heads in 2-byte accesses, q and k in a launch each: 12.5 +
// 4.9 us at 986 rows of 28 + 4 heads, 65.7 + 13.5 us at 16512; now 6.9 and 44.9.
constexpr int kRopeRows = 4;
constexpr int kRopeMaxHalf = 128;
struct RopeTensors {
  __bf16 *x[2];
  int heads[2];
  int64_t stride[2];  // elements
};
__global__ __launch_bounds__(kRowThreads) void rope_rows_kernel(int64_t rows, int d, const RopeTensors t,
                                                                const int32_t *pos, double log2_theta) {
  __shared__ float sn[kRopeRows][kRopeMaxHalf], cs[kRopeRows][kRopeMaxHalf];
  const int half = d / 2, pieces = half / 8;
  const int64_t row0 = (int64_t)blockIdx.x * kRopeRows;
  const int n_rows = (int)min((int64_t)kRopeRows, rows - row0);
  for (int w = threadIdx.x; w < n_rows * half; w += kRowThreads) {
    const int r = w / half, i = w - r * half;
    const double inv = exp2(-(2.0 * i / d) * log2_theta);
    double sd, cd;
    sincos((double)pos[row0 + r] * inv, &sd, &cd);
    sn[r][i] = (float)sd;
    cs[r][i] = (float)cd;
  }
  __syncthreads();
  const int heads = t.heads[0] + t.heads[1], items = n_rows * heads * pieces;
  for (int w = threadIdx.x; w < items; w += kRowThreads) {
    const int c = w % pieces, hr = w / pieces, h = hr % heads, r = hr / heads;
    const int k = h < t.heads[0] ? 0 : 1;
    __bf16 *p = t.x[k] + (row0 + r) * t.stride[k] + (int64_t)(h - (k ? t.heads[0] : 0)) * d + 8 * c;
    const bf16x8 a = *reinterpret_cast<const bf16x8 *>(p), b = *reinterpret_cast<const bf16x8 *>(p + half);
    bf16x8 oa, ob;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float s = sn[r][8 * c + e], co = cs[r][8 * c + e], x = (float)a[e], y = (float)b[e];
      oa[e] = (__bf16)(x * co - y * s);
      ob[e] = (__bf16)(y * co + x * s);
    }
    *reinterpret_cast<bf16x8 *>(p) = oa;
    *reinterpret_cast<bf16x8 *>(p + half) = ob;
  }
}

// The same for few heads, and for head sizes, strides or addresses that do not
// allow 16-byte pieces: one thread per (row, i) rotates pair i of every head.
__global__ __launch_bounds__(kRowThreads) void rope_kernel(int64_t rows, int heads, int d, int64_t row_stride,
                                                           __bf16 *x, const int32_t *pos, double log2_theta) {
  const int half = d / 2;
  const int64_t t = (int64_t)blockIdx.x * kRowThreads + threadIdx.x;
  if (t >= rows * half) return;
  const int64_t row = t / half;
  const int i = (int)(t - row * half);
  const double inv = exp2(-(2.0 * i / d) * log2_theta);
  double sd, cd;
  sincos((double)pos[row] * inv, &sd, &cd);
  const float s = (float)sd, c = (float)cd;
  __bf16 *p = x + row * row_stride + i;
  for (int h = 0; h < heads; ++h, p += d) {
    const float a = (float)p[0], b = (float)p[half];
    p[0] = (__bf16)(a * c - b * s);
    p[half] = (__bf16)(b * c + a * s);
  }
}

// out[r][j] = SiLU(gu[r][j]) * gu[r][width + j] (gate then up in one row).
__global__ __launch_bounds__(kRowThreads) void silu_mul_kernel(int64_t rows, int width, const __bf16 *gu,
                                                               __bf16 *out) {
  const int pieces = width / 8;
  const int64_t t = (int64_t)blockIdx.x * kRowThreads + threadIdx.x;
  if (t >= rows * pieces) return;
  const int64_t row = t / pieces;
  const int j = (int)(t - row * pieces);
  const bf16x8 g = reinterpret_cast<const bf16x8 *>(gu + row * 2 * width)[j];
  const bf16x8 u = reinterpret_cast<const bf16x8 *>(gu + row * 2 * width + width)[j];
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float gf = (float)g[e];
    o[e] = (__bf16)(gf / (1.0f + __expf(-gf)) * (float)u[e]);
  }
  reinterpret_cast<bf16x8 *>(out + row * width)[j] = o;
}

}  // namespace

hipError_t launch_rmsnorm(int64_t rows, int width, const void *x, const void *w, float eps, void *y,
                          hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  const int64_t blocks = (rows + kRowThreads / 64 - 1) / (kRowThreads / 64);
  rmsnorm_kernel<<<dim3((unsigned)blocks), dim3(kRowThreads), 0, st>>>(
      rows, width, static_cast<const __bf16 *>(x), static_cast<const __bf16 *>(w), eps, static_cast<__bf16 *>(y));
  return hipGetLastError();
}

hipError_t launch_rope(int64_t rows, int heads, int d, int64_t row_stride, void *x, const int32_t *pos,
                       double theta, hipStream_t st, int heads2, int64_t row_stride2, void *x2) {
  if (rows <= 0 || heads <= 0) return hipSuccess;
  // 16-byte pieces of a half head: every piece of either tensor aligned
  auto whole = [&](const void *p, int64_t stride) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && stride % 8 == 0; };
  // and enough of them per row to share its sines: one tensor with at most 8 heads
  // of 512 features in all takes a thread per pair (32896 rows, pieces and threads:
  // 1 x 64 10.7 and 7.5 us, 8 x 64 14.9 and 13.6, 4 x 128 17.9 and 16.2; 100000 rows
  // of 4 x 16 21.7 and 8.8); with more heads that thread is the longer way (5043 rows
  // of 16 x 32 4.5 and 5.7, 28 x 128 12 and 16), and two tensors would be two launches
  const bool few = !x2 && heads <= 8 && heads * d <= 512;
  if (!few && d % 16 == 0 && d / 2 <= kRopeMaxHalf && whole(x, row_stride) && (!x2 || whole(x2, row_stride2))) {
    const RopeTensors t{{static_cast<__bf16 *>(x), static_cast<__bf16 *>(x2)}, {heads, x2 ? heads2 : 0},
                        {row_stride, row_stride2}};
    rope_rows_kernel<<<dim3((unsigned)((rows + kRopeRows - 1) / kRopeRows)), dim3(kRowThreads), 0, st>>>(
        rows, d, t, pos, log2(theta));
    return hipGetLastError();
  }
  const int64_t n = rows * (d / 2);
  const dim3 grid((unsigned)((n + kRowThreads - 1) / kRowThreads));
  rope_kernel<<<grid, dim3(kRowThreads), 0, st>>>(rows, heads, d, row_stride, static_cast<__bf16 *>(x), pos,
                                                  log2(theta));
  if (x2)
    rope_kernel<<<grid, dim3(kRowThreads), 0, st>>>(rows, heads2, d, row_stride2, static_cast<__bf16 *>(x2), pos,
                                                    log2(theta));
  return hipGetLastError();
}

hipError_t launch_silu_mul(int64_t rows, int width, const void *gu, void *out, hipStream_t st) {
  const int64_t n = rows * (width / 8);
  if (n <= 0) return hipSuccess;
  silu_mul_kernel<<<dim3((unsigned)((n + kRowThreads - 1) / kRowThreads)), dim3(kRowThreads), 0, st>>>(
      rows, width, static_cast<const __bf16 *>(gu), static_cast<__bf16 *>(out));
  return hipGetLastError();
}

}  // namespace daf
