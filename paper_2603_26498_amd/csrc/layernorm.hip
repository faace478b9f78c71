// LayerNorm (or RMSNorm) over the last dimension, one wavefront per row (gfx950, wave64).
//
// The row (fp32) is read once with 16-byte loads and kept in registers; the
// mean and the centred sum of squares are reduced across the wave in fp32 (two
// passes over registers, no second trip to memory); the result is written as
// bf16 or fp32.  HBM-bound: 4*d bytes read + 2*d (or 4*d) bytes written per row.
// The loads of a row are requested together, at clamped indices instead of under a condition, and gamma and beta are not
// read column group by column group behind the stores of the group before (1280 wide: 256 rows 4.7 -> 3.7 us, 16656 rows
// 23.3 -> 21.8).  Without the scheduling barrier behind them the compiler moves those of gamma and beta behind the first
// reduction, which exposes one more memory round trip; the reductions stay on the vector ALU (wave_sum).  4096 x 1280
// 7.3 -> 6.7 us; a pass over 256 tokens (64 norms behind sliced products) 1912 -> 1884.
#include "tcmv_internal.h"
#include "device_utils.h"

namespace tcmv {

// Sum of the squares of four values, the products paired in one written-out way: left to the compiler, the pairing (and
// with it the last bit of the sum) changes with the code around it.
__device__ __forceinline__ float square_sum(const float4& v) { return fmaf(v.x, v.x, v.y * v.y) + fmaf(v.z, v.z, v.w * v.w); }

template <int NV, bool OUT_BF16, bool RMS>
__global__ __launch_bounds__(256) void layernorm_kernel(const float* x, const float* __restrict__ gamma,
                                                        const float* __restrict__ beta, void* y,
                                                        int64_t rows, int d, float eps) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int nvec = d >> 2;
  const float4* xr = reinterpret_cast<const float4*>(x + row * d);
  const float4* g4 = reinterpret_cast<const float4*>(gamma);
  const float4* b4 = reinterpret_cast<const float4*>(beta);
  float4 v[NV], g[NV], b[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) v[j] = xr[min(lane + 64 * j, nvec - 1)];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int i = min(lane + 64 * j, nvec - 1);
    g[j] = g4[i];
    b[j] = RMS ? make_float4(0.f, 0.f, 0.f, 0.f) : b4[i];
  }
  __builtin_amdgcn_sched_barrier(0);
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) s += lane + 64 * j < nvec ? (v[j].x + v[j].y) + (v[j].z + v[j].w) : 0.f;
  const float mean = RMS ? 0.f : wave_sum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    v[j].x -= mean; v[j].y -= mean; v[j].z -= mean; v[j].w -= mean;
    q += lane + 64 * j < nvec ? square_sum(v[j]) : 0.f;
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + eps);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    float4 o;
    o.x = v[j].x * rstd * g[j].x + b[j].x;
    o.y = v[j].y * rstd * g[j].y + b[j].y;
    o.z = v[j].z * rstd * g[j].z + b[j].z;
    o.w = v[j].w * rstd * g[j].w + b[j].w;
    const int i = lane + 64 * j;
    if (i < nvec) {
      if (OUT_BF16) {
        uint2 p;
        p.x = pack_bf16x2(o.x, o.y);
        p.y = pack_bf16x2(o.z, o.w);
        reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(y) + row * d)[i] = p;
      } else {
        reinterpret_cast<float4*>(reinterpret_cast<float*>(y) + row * d)[i] = o;
      }
    }
  }
}

template <bool OUT_BF16, bool RMS>
static hipError_t launch_ln_t(const float* x, const float* g, const float* b, void* y, int64_t rows, int d, float eps,
                              hipStream_t s) {
  dim3 grid((unsigned)((rows + 3) / 4)), block(256);
  const int nv = (d / 4 + 63) / 64;
#define TCMV_LN_CASE(N)                                                                                   \
  case N:                                                                                                 \
    hipLaunchKernelGGL((layernorm_kernel<N, OUT_BF16, RMS>), grid, block, 0, s, x, g, b, y, rows, d, eps); \
    break;
  switch (nv) {
    TCMV_LN_CASE(1) TCMV_LN_CASE(2) TCMV_LN_CASE(3) TCMV_LN_CASE(4)
    TCMV_LN_CASE(5) TCMV_LN_CASE(6) TCMV_LN_CASE(7) TCMV_LN_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef TCMV_LN_CASE
  return hipGetLastError();
}

// The same over rows that are first completed by the four fp32 partial sums of the product before (bias + slice 0 + .. +
// slice 3, the order of the separate reduction): saves that kernel's launch and its trip through x.  Requests come here
// whose products are cut along k, at 1280 columns up to 580 rows behind the out-projection and up to 1550 behind fc2: bound
// by latency and, towards the upper end, by the slices (1120 rows 7.6 us).  A row gets a workgroup of its own and
// everything it needs, gamma and beta too, is requested before anything is used.  256 x 1280: 4.3 us against 4.4 + 4.7 in
// two kernels (11.3 with a wavefront per row).
template <int NV, bool OUT_BF16, bool RMS>
__global__ __launch_bounds__(256) void layernorm_slices_kernel(float* x, const float* __restrict__ partial,
                                                               const float* __restrict__ bias, const float* __restrict__ gamma,
                                                               const float* __restrict__ beta, void* y,
                                                               int64_t rows, int d, float eps) {
  __shared__ float sums[2][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = blockIdx.x;
  const int nvec = d >> 2;
  float4* xr = reinterpret_cast<float4*>(x + row * d);
  float4 v[NV], acc[NV], p[4][NV], g[NV], b[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int i = min(tid + 256 * j, nvec - 1);      // no branches: a load under a condition is not kept whole
    v[j] = xr[i];
    acc[j] = reinterpret_cast<const float4*>(bias)[i];
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) p[sl][j] = reinterpret_cast<const float4*>(partial + ((size_t)sl * rows + row) * d)[i];
    g[j] = reinterpret_cast<const float4*>(gamma)[i];
    b[j] = RMS ? make_float4(0.f, 0.f, 0.f, 0.f) : reinterpret_cast<const float4*>(beta)[i];
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) { acc[j].x += p[sl][j].x; acc[j].y += p[sl][j].y; acc[j].z += p[sl][j].z; acc[j].w += p[sl][j].w; }
    v[j].x += acc[j].x; v[j].y += acc[j].y; v[j].z += acc[j].z; v[j].w += acc[j].w;
    const bool ok = tid + 256 * j < nvec;
    if (OUT_BF16 && ok) xr[tid + 256 * j] = v[j];
    s += ok ? (v[j].x + v[j].y) + (v[j].z + v[j].w) : 0.f;
  }
  float mean = 0.f;
  if (!RMS) {
    s = wave_sum(s);
    if (lane == 0) sums[0][wave] = s;
    __syncthreads();
    mean = ((sums[0][0] + sums[0][1]) + (sums[0][2] + sums[0][3])) / (float)d;
  }
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j)
    if (tid + 256 * j < nvec) {
      v[j].x -= mean; v[j].y -= mean; v[j].z -= mean; v[j].w -= mean;
      q += square_sum(v[j]);
    }
  q = wave_sum(q);
  if (lane == 0) sums[1][wave] = q;
  __syncthreads();
  const float rstd = 1.0f / sqrtf(((sums[1][0] + sums[1][1]) + (sums[1][2] + sums[1][3])) / (float)d + eps);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int i = tid + 256 * j;
    if (i < nvec) {
      float4 o;
      o.x = v[j].x * rstd * g[j].x + b[j].x;
      o.y = v[j].y * rstd * g[j].y + b[j].y;
      o.z = v[j].z * rstd * g[j].z + b[j].z;
      o.w = v[j].w * rstd * g[j].w + b[j].w;
      if (OUT_BF16) {
        uint2 pk;
        pk.x = pack_bf16x2(o.x, o.y);
        pk.y = pack_bf16x2(o.z, o.w);
        reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(y) + row * d)[i] = pk;
      } else {
        reinterpret_cast<float4*>(reinterpret_cast<float*>(y) + row * d)[i] = o;
      }
    }
  }
}

// Reference for the bandwidth-bound kernels: n_in 16-byte words read once, n_out 16-byte words written once, no
// other work - what a kernel that moves these bytes can reach at best at this size.
__global__ __launch_bounds__(256) void stream_ref_kernel(const uint4* __restrict__ in, uint4* __restrict__ out,
                                                         size_t n_in, size_t n_out) {
  const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x, nt = (size_t)gridDim.x * 256;
  uint4 acc = {0u, 0u, 0u, 0u};
  for (size_t i = tid; i < n_in; i += nt) {
    const uint4 v = in[i];
    acc.x ^= v.x; acc.y ^= v.y; acc.z ^= v.z; acc.w ^= v.w;
  }
  for (size_t i = tid; i < n_out; i += nt) out[i] = acc;
}

hipError_t launch_stream_ref(const void* in, size_t in_bytes, void* out, size_t out_bytes, hipStream_t s) {
  if (in_bytes % 16 || out_bytes % 16 || reinterpret_cast<uintptr_t>(in) % 16 || reinterpret_cast<uintptr_t>(out) % 16)
    return hipErrorInvalidValue;
  if (in_bytes + out_bytes == 0) return hipSuccess;
  hipLaunchKernelGGL(stream_ref_kernel, dim3(2048), dim3(256), 0, s, reinterpret_cast<const uint4*>(in),
                     reinterpret_cast<uint4*>(out), in_bytes / 16, out_bytes / 16);
  return hipGetLastError();
}

hipError_t launch_layernorm(const float* x, const float* g, const float* b, void* y, int64_t rows, int d, float eps,
                            int out_bf16, hipStream_t s, int rms) {
  if (rows == 0) return hipSuccess;
  if (d % 4 || d <= 0 || d > 2048) return hipErrorInvalidValue;
  if (rms) return out_bf16 ? launch_ln_t<true, true>(x, g, b, y, rows, d, eps, s) : launch_ln_t<false, true>(x, g, b, y, rows, d, eps, s);
  return out_bf16 ? launch_ln_t<true, false>(x, g, b, y, rows, d, eps, s) : launch_ln_t<false, false>(x, g, b, y, rows, d, eps, s);
}

template <bool OUT_BF16, bool RMS>
static hipError_t launch_ln_slices_t(float* x, const float* partial, const float* bias, const float* g, const float* b, void* y,
                                     int64_t rows, int d, float eps, hipStream_t s) {
  const dim3 grid((unsigned)rows), block(256);
  if (d <= 1024) hipLaunchKernelGGL((layernorm_slices_kernel<1, OUT_BF16, RMS>), grid, block, 0, s, x, partial, bias, g, b, y, rows, d, eps);
  else hipLaunchKernelGGL((layernorm_slices_kernel<2, OUT_BF16, RMS>), grid, block, 0, s, x, partial, bias, g, b, y, rows, d, eps);
  return hipGetLastError();
}

hipError_t launch_layernorm_slices(float* x, const float* partial, const float* bias, const float* g, const float* b, void* y,
                                   int64_t rows, int d, float eps, int out_bf16, hipStream_t s, int rms) {
  if (rows == 0) return hipSuccess;
  if (d % 4 || d <= 0 || d > 2048 || !partial || !bias || (!out_bf16 && y != x)) return hipErrorInvalidValue;
  if (rms) return out_bf16 ? launch_ln_slices_t<true, true>(x, partial, bias, g, b, y, rows, d, eps, s)
                           : launch_ln_slices_t<false, true>(x, partial, bias, g, b, y, rows, d, eps, s);
  return out_bf16 ? launch_ln_slices_t<true, false>(x, partial, bias, g, b, y, rows, d, eps, s)
                  : launch_ln_slices_t<false, false>(x, partial, bias, g, b, y, rows, d, eps, s);
}

}  // namespace tcmv
