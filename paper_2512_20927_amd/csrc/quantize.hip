// Storage encoders for the feature table: bfloat16 and OCP FP8 e4m3 with a
// per-Gaussian float32 scale. Both renderers decode these in their load path
// and accumulate in float32. Both encoders are bound by HBM: the float32
// table read once, the codes written once.
#include "common.h"

namespace qr {

// float32 -> bfloat16 bits, round to nearest, ties to even.
__device__ __forceinline__ uint16_t f32_to_bf16(float x) {
  const uint32_t b = __float_as_uint(x);
  return static_cast<uint16_t>((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
}

// |x| <= 448 (finite) -> e4m3 code, nearest with ties to even.
// Normal range: round the float32 pattern to 3 mantissa bits (the carry may
// bump the exponent) and rebias the exponent from 127 to 7. Below 2^-6 the
// e4m3 grid is uniform with step 2^-9, so the code is rint(|x| * 2^9).
__device__ __forceinline__ uint32_t f32_to_e4m3(float x) {
  const uint32_t sign = (__float_as_uint(x) >> 24) & 0x80u;
  const float mag = fminf(fabsf(x), 448.f);
  uint32_t code;
  if (mag < 0.015625f) {
    code = static_cast<uint32_t>(rintf(mag * 512.f));
  } else {
    const uint32_t b = __float_as_uint(mag);
    const uint32_t r = (b + 0x7FFFFu + ((b >> 20) & 1u)) >> 20;
    code = r - (120u << 3);
  }
  return sign | code;
}

// Eight elements per thread: two 16-byte loads, one 16-byte store; the last,
// fewer than eight, by the threads after them. (1M x 512: 1,012 -> 522 us against
// the element-wise kernel below.)
__global__ void __launch_bounds__(256)
quantize_bf16_vec_kernel(int64_t count, const float4* __restrict__ f, uint4* __restrict__ out) {
  const int64_t i = blockIdx.x * 256LL + threadIdx.x, count8 = count >> 3;
  if (i >= count8) {
    const int64_t e = 7 * count8 + i;  // 8 count8 + (i - count8)
    if (e < count) reinterpret_cast<uint16_t*>(out)[e] = f32_to_bf16(reinterpret_cast<const float*>(f)[e]);
    return;
  }
  const float4 a = f[2 * i], b = f[2 * i + 1];
  const auto pair = [](float x, float y) {
    return static_cast<uint32_t>(f32_to_bf16(x)) | (static_cast<uint32_t>(f32_to_bf16(y)) << 16);
  };
  out[i] = make_uint4(pair(a.x, a.y), pair(a.z, a.w), pair(b.x, b.y), pair(b.z, b.w));
}

__global__ void __launch_bounds__(256)
quantize_bf16_kernel(int64_t count, const float* __restrict__ f, uint16_t* __restrict__ out) {
  const int64_t i = blockIdx.x * 256LL + threadIdx.x;
  if (i < count) out[i] = f32_to_bf16(f[i]);
}

// Codes of four values (byte 0 first): sign | hardware conversion of the
// magnitude, clamped to 448 (v_cvt_pk_fp8_f32 rounds to nearest even onto the
// OCP e4m3 grid, subnormals included: the codes of f32_to_e4m3).
__device__ __forceinline__ uint32_t f32x4_to_e4m3(float4 v) {
  const float m0 = fminf(fabsf(v.x), 448.f), m1 = fminf(fabsf(v.y), 448.f);
  const float m2 = fminf(fabsf(v.z), 448.f), m3 = fminf(fabsf(v.w), 448.f);
  int r = __builtin_amdgcn_cvt_pk_fp8_f32(m0, m1, 0, false);
  r = __builtin_amdgcn_cvt_pk_fp8_f32(m2, m3, r, true);
  const uint32_t sign = ((__float_as_uint(v.x) >> 24) & 0x80u) | ((__float_as_uint(v.y) >> 16) & 0x8000u) |
                        ((__float_as_uint(v.z) >> 8) & 0x800000u) | (__float_as_uint(v.w) & 0x80000000u);
  return sign | static_cast<uint32_t>(r);
}

// Rows of whole float4s up to V * 256 wide, held in registers: lpr lanes per
// row (a power of two, so a wave takes 64 / lpr rows side by side), V float4s
// per lane, kRows such groups of rows per wave with all their loads requested
// before the first is used; each row is read once and written as 4-byte
// codes. (1M x 512: 1,100 -> 453 us against the kernel below, which reads the
// row twice in 4-byte and writes it in 1-byte pieces: 5.7 TB/s; 4.7 is a
// large copy's rate.)
constexpr int kQuantRows = 2;

template <int V>
__global__ void __launch_bounds__(256)
quantize_e4m3_rows_kernel(int64_t n, int dim4, int lpr_log, const float4* __restrict__ f,
                          uint32_t* __restrict__ out, float* __restrict__ scale) {
  const int lane = threadIdx.x & 63;
  const int rpw = 64 >> lpr_log;  // rows of a group
  const int c = lane & ((1 << lpr_log) - 1);
  const int64_t row0 = (blockIdx.x * 4LL + (threadIdx.x >> 6)) * (rpw * kQuantRows) + (lane >> lpr_log);
  float4 x[kQuantRows][V];
#pragma unroll
  for (int r = 0; r < kQuantRows; ++r) {
    const int64_t row = row0 + r * rpw;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int col = c + (v << lpr_log);
      x[r][v] = row < n && col < dim4 ? f[row * dim4 + col] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
#pragma unroll
  for (int r = 0; r < kQuantRows; ++r) {
    const int64_t row = row0 + r * rpw;
    float m = 0.f;
#pragma unroll
    for (int v = 0; v < V; ++v)
      m = fmaxf(m, fmaxf(fmaxf(fabsf(x[r][v].x), fabsf(x[r][v].y)), fmaxf(fabsf(x[r][v].z), fabsf(x[r][v].w))));
    for (int off = (1 << lpr_log) >> 1; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    const float s = m > 0.f ? m / 448.f : 1.f;
    if (row >= n) continue;
    if (c == 0) scale[row] = s;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int col = c + (v << lpr_log);
      if (col < dim4)
        out[row * dim4 + col] = f32x4_to_e4m3(make_float4(x[r][v].x / s, x[r][v].y / s, x[r][v].z / s, x[r][v].w / s));
    }
  }
}

// Any width and alignment: one wave64 per row, max |f| -> scale, then the
// codes of f / scale
__global__ void __launch_bounds__(256)
quantize_e4m3_kernel(int64_t n, int dim, const float* __restrict__ f, uint8_t* __restrict__ out,
                     float* __restrict__ scale) {
  const int lane = threadIdx.x & 63;
  const int64_t row = blockIdx.x * 4LL + (threadIdx.x >> 6);
  if (row >= n) return;
  const float* fr = f + row * dim;
  float m = 0.f;
  for (int d = lane; d < dim; d += 64) m = fmaxf(m, fabsf(fr[d]));
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  const float s = m > 0.f ? m / 448.f : 1.f;
  if (lane == 0) scale[row] = s;
  uint8_t* orow = out + row * dim;
  for (int d = lane; d < dim; d += 64) orow[d] = static_cast<uint8_t>(f32_to_e4m3(fr[d] / s));
}

}  // namespace qr

using namespace qr;

extern "C" int qr_quantize_features(void* stream, int64_t n, int32_t dim, const float* features,
                                    int32_t dtype, void* out, float* scale) {
  if (n < 0 || dim <= 0) return fail(QR_ERR_INVALID_ARG, "qr_quantize_features: bad sizes");
  if (dtype != QR_BF16 && dtype != QR_FP8_E4M3)
    return fail(QR_ERR_UNSUPPORTED, "qr_quantize_features: dtype must be QR_BF16 or QR_FP8_E4M3");
  if (n == 0) return QR_OK;
  if (!features || !out) return fail(QR_ERR_INVALID_ARG, "qr_quantize_features: null pointer");
  if (dtype == QR_FP8_E4M3 && !scale)
    return fail(QR_ERR_INVALID_ARG, "qr_quantize_features: FP8 needs a scale array");
  hipStream_t s = as_stream(stream);
  // The vector kernels need their accesses aligned: the float4 rows and the
  // code words of e4m3 (widths of whole float4s, up to the 1,024 that fit in
  // registers), eight-element pieces of the whole table for bfloat16.
  const auto aligned = [](const void* p, size_t a) { return reinterpret_cast<uintptr_t>(p) % a == 0; };
  if (dtype == QR_BF16) {
    const int64_t count = n * dim;
    if (aligned(features, 16) && aligned(out, 16))
      hipLaunchKernelGGL(quantize_bf16_vec_kernel, dim3(static_cast<unsigned>(ceil_div(count / 8 + count % 8, 256))),
                         dim3(256), 0, s, count, reinterpret_cast<const float4*>(features),
                         reinterpret_cast<uint4*>(out));
    else
      hipLaunchKernelGGL(quantize_bf16_kernel, dim3(static_cast<unsigned>(ceil_div(count, 256))),
                         dim3(256), 0, s, count, features, static_cast<uint16_t*>(out));
  } else if (dim % 4 == 0 && dim <= 1024 && aligned(features, 16) && aligned(out, 4)) {
    const int dim4 = dim / 4;
    int lpr_log = 0;
    while (lpr_log < 6 && (1 << lpr_log) < dim4) ++lpr_log;
    const int64_t rows = 4LL * kQuantRows * (64 >> lpr_log);  // of a workgroup
#define QR_LAUNCH(V)                                                                                    \
  hipLaunchKernelGGL(quantize_e4m3_rows_kernel<V>, dim3(static_cast<unsigned>(ceil_div(n, rows))),      \
                     dim3(256), 0, s, n, dim4, lpr_log, reinterpret_cast<const float4*>(features),      \
                     static_cast<uint32_t*>(out), scale)
    if (dim4 <= 64) QR_LAUNCH(1);
    else if (dim4 <= 128) QR_LAUNCH(2);
    else QR_LAUNCH(4);
#undef QR_LAUNCH
  } else {
    hipLaunchKernelGGL(quantize_e4m3_kernel, dim3(static_cast<unsigned>(ceil_div(n, 4))), dim3(256),
                       0, s, n, dim, features, static_cast<uint8_t*>(out), scale);
  }
  return check_launch("qr_quantize_features");
}
