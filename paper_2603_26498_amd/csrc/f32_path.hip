// fp32 kernels: GEMM with the same epilogues as the bf16 one, and attention, both on the fp32
// matrix instructions (true fp32 multiply-adds: v_mfma_f32_16x16x4_f32, v_mfma_f32_32x32x2_f32).
//
// An MFMA does not care which k-index a lane holds as long as both operands agree, so everywhere
// below a lane owns CONSECUTIVE k-elements (16-byte loads) and the instruction of step s takes
// element s of every lane's run.
#include "tcmv_internal.h"
#include "device_utils.h"

namespace tcmv {

namespace {
typedef __attribute__((ext_vector_type(4))) float f32v4;
typedef f32v4 __attribute__((aligned(4))) f32v4_mem;   // rows need not be 16-byte aligned
}  // namespace

// one output value: bias, epilogue, store
template <int EPI>
__device__ __forceinline__ void store_f32(const GemmArgs& g, int64_t row, int col, float val) {
  if (g.bias) val += g.bias[col];
  float* C = reinterpret_cast<float*>(g.c);
  if (EPI == EPI_STORE || EPI == EPI_QKV) {
    C[(size_t)row * g.ldc + col] = val;
  } else if (EPI == EPI_GELU) {
    C[(size_t)row * g.ldc + col] = gelu_erf(val);
  } else if (EPI == EPI_RESID) {
    C[(size_t)row * g.ldc + col] += val;
  } else if (EPI == EPI_EMBED) {
    const int pi = g.pos_idx ? g.pos_idx[row] : 0;
    if (g.pos_kind == 1) {
      val += g.pos0[(size_t)pi * g.n + col];
    } else if (g.pos_kind == 2) {
      val += g.pos0[(size_t)(pi & 0xFFFF) * g.n + col] + g.pos1[(size_t)(pi >> 16) * g.n + col];
    }
    const int64_t dst = g.dst_row ? (int64_t)g.dst_row[row] : row;
    C[(size_t)dst * g.ldc + col] = val;
  }
}

// ---------------------------------------------------------------------------
// Few output tiles (one small request): a 16x16 tile per workgroup, the contraction dealt out to
// its four waves in chunks of 16, no staging (operands go straight from the caches to registers,
// all loads of four chunks in flight together), partial sums added through LDS in wave order.
// Such a product is bound by latency, not by arithmetic: what counts is many workgroups and one
// memory round trip.  197 rows, one layer's products: 3 - 8 us each in a pass (35 - 85 us with 64x64 tiles on the
// vector ALU).
// ---------------------------------------------------------------------------
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(GemmArgs g) {
  __shared__ float part[4][16][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * 16;
  const int n0 = blockIdx.x * 16;
  int64_t ra = m0 + lr;
  if (ra > g.m - 1) ra = g.m - 1;
  const int rw = min(n0 + lr, g.n - 1);
  const float* A = reinterpret_cast<const float*>(g.a) + (size_t)ra * g.lda + 4 * lg;
  const float* W = reinterpret_cast<const float*>(g.w) + (size_t)rw * g.k + 4 * lg;
  const int nc = g.k >> 4;
  f32v4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;
  for (int c = wave; c < nc; c += 4 * U) {
    f32v4 a[U], w[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + 4 * u < nc) {
        a[u] = *reinterpret_cast<const f32v4_mem*>(A + (size_t)(c + 4 * u) * 16);
        w[u] = *reinterpret_cast<const f32v4_mem*>(W + (size_t)(c + 4 * u) * 16);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + 4 * u < nc)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][s], w[u][s], acc, 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) part[wave][4 * lg + v][lr] = acc[v];
  __syncthreads();
  const int r = tid >> 4, c = tid & 15;
  if (m0 + r < g.m && n0 + c < g.n)
    store_f32<EPI>(g, m0 + r, n0 + c, (part[0][r][c] + part[1][r][c]) + (part[2][r][c] + part[3][r][c]));
}

// ---------------------------------------------------------------------------
// Larger products: 64x64 tiles, four waves of 32x32, k-slices of 32 staged in LDS (rows padded to 36
// floats), the next slice on its way into registers while the current one is multiplied.
// 3152 x 1024 x 256: 22.9 us, 72 TFLOP/s (the fp32 matrix rate is 157).  VEC: k is a multiple of 4; otherwise element-wise loads.
// ---------------------------------------------------------------------------
template <int EPI, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  constexpr int BT = 64, BK = 32, STR = BK + 4;
  __shared__ __attribute__((aligned(16))) float sa[BT * STR], sb[BT * STR];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lg = lane >> 5;
  const int64_t m0 = (int64_t)blockIdx.y * BT;
  const int n0 = blockIdx.x * BT;
  // thread -> rows tid/8 and tid/8 + 32 of the slice, k-elements 4*(tid%8) .. +3
  const int tr = tid >> 3, tk = (tid & 7) * 4;
  const float* pa[2];
  const float* pb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int64_t ra = m0 + tr + 32 * i;
    if (ra > g.m - 1) ra = g.m - 1;
    pa[i] = reinterpret_cast<const float*>(g.a) + (size_t)ra * g.lda;
    pb[i] = reinterpret_cast<const float*>(g.w) + (size_t)min(n0 + tr + 32 * i, g.n - 1) * g.k;
  }
  auto load4 = [&](const float* p, int k) {
    f32v4 v = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
      if (k < g.k) v = *reinterpret_cast<const f32v4_mem*>(p + k);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j < g.k) v[j] = p[k + j];
    }
    return v;
  };
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  f32v4 na[2], nb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) { na[i] = load4(pa[i], tk); nb[i] = load4(pb[i], tk); }
  const float* fa = sa + ((wave >> 1) * 32 + lr) * STR + lg * 16;
  const float* fb = sb + ((wave & 1) * 32 + lr) * STR + lg * 16;
  for (int k0 = 0; k0 < g.k; k0 += BK) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *reinterpret_cast<f32v4*>(sa + (tr + 32 * i) * STR + tk) = na[i];
      *reinterpret_cast<f32v4*>(sb + (tr + 32 * i) * STR + tk) = nb[i];
    }
    __syncthreads();
    if (k0 + BK < g.k)
#pragma unroll
      for (int i = 0; i < 2; ++i) { na[i] = load4(pa[i], k0 + BK + tk); nb[i] = load4(pb[i], k0 + BK + tk); }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32v4 a = *reinterpret_cast<const f32v4*>(fa + 4 * q), b = *reinterpret_cast<const f32v4*>(fb + 4 * q);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], b[s], acc, 0, 0, 0);
    }
  }
  const int col = n0 + (wave & 1) * 32 + lr;
  if (col >= g.n) return;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t row = m0 + (wave >> 1) * 32 + 8 * (v >> 2) + 4 * lg + (v & 3);
    if (row < g.m) store_f32<EPI>(g, row, col, acc[v]);
  }
}

template <int EPI>
static hipError_t launch_gemm_f32_t(const GemmArgs& a, hipStream_t s) {
  const int64_t ty = (a.m + 63) / 64, tx = (a.n + 63) / 64;
  // Up to about 100 64x64 tiles (a third of the CUs) the 16x16 tiles win, k = 256 / 1024: 48 tiles 4.8 against 8.4 us,
  // 28 tiles 9.1 against 26.1 us, 100 tiles 8.2 against 8.6 / 26.9 against 26.3 us; 208 tiles 13.7 against 8.7 us.
  if (a.k % 16 == 0 && tx * ty <= 100) {
    hipLaunchKernelGGL((gemm_f32_small_kernel<EPI>), dim3((unsigned)((a.n + 15) / 16), (unsigned)((a.m + 15) / 16)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  if (ty > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)tx, (unsigned)ty);
  if (a.k % 4 == 0) hipLaunchKernelGGL((gemm_f32_kernel<EPI, true>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((gemm_f32_kernel<EPI, false>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  if (a.m == 0 || a.n == 0) return hipSuccess;
  if (a.k <= 0) return hipErrorInvalidValue;
  switch (a.epi) {
    case EPI_STORE: return launch_gemm_f32_t<EPI_STORE>(a, s);
    case EPI_GELU: return launch_gemm_f32_t<EPI_GELU>(a, s);
    case EPI_RESID: return launch_gemm_f32_t<EPI_RESID>(a, s);
    case EPI_EMBED: return launch_gemm_f32_t<EPI_EMBED>(a, s);
    case EPI_QKV: return launch_gemm_f32_t<EPI_QKV>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------------------
// Attention, fp32: a workgroup of four waves handles 16 query rows of one segment and one head; the
// tiles of 16 keys are dealt out to the waves, each keeps its own online softmax, and the four
// partial results meet in LDS.  S^T = K Q^T leaves a lane with one query (lane & 15) and four keys
// (4 * (lane >> 4) + v), which is the B operand of O^T += V^T P^T as it stands.  A small request is bound by
// latency: 197 tokens, 4 heads of 64 are 52 workgroups of four waves with at most four key tiles each (9.6 us;
// 273 us with one thread per query walking all keys).
// ---------------------------------------------------------------------------
template <int DH>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a) {
  constexpr int BQ = kAttnBQ_f32, ND = DH / 16;
  static_assert(BQ == 16, "one 16x16 tile of queries");
  __shared__ float so[4][BQ][DH + 4];
  __shared__ float sm[4][BQ], sl[4][BQ];
  const int head = blockIdx.y;
  const AttnWork w = a.work[blockIdx.x];
  const float* K = reinterpret_cast<const float*>(a.k) + head * DH;
  const float* V = reinterpret_cast<const float*>(a.v) + head * DH;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  // a lane holds dimensions lg * DH/4 .. of its query and key rows
  f32v4 q[ND], o[ND];
  {
    const float* qp = reinterpret_cast<const float*>(a.q) + (size_t)(w.q0 + min(lr, w.nq - 1)) * a.ldqk + head * DH + lg * (DH / 4);
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      q[i] = *reinterpret_cast<const f32v4_mem*>(qp + 4 * i) * a.scale;
      o[i] = f32v4{0.f, 0.f, 0.f, 0.f};
    }
  }
  float m = -INFINITY, l = 0.f;
  for (int j0 = __builtin_amdgcn_readfirstlane(wave) * 16; j0 < w.seg_len; j0 += 64) {      // scalar: so are its conditions
    const float* kp = K + (size_t)(w.seg_start + min(j0 + lr, w.seg_len - 1)) * a.ldqk + lg * (DH / 4);
    f32v4 kf[ND];
    float vf[4][ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) kf[i] = *reinterpret_cast<const f32v4_mem*>(kp + 4 * i);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float* vp = V + (size_t)(w.seg_start + min(j0 + 4 * lg + v, w.seg_len - 1)) * a.ldv + lr;
#pragma unroll
      for (int i = 0; i < ND; ++i) vf[v][i] = vp[16 * i];
    }
    if (j0 + 16 > w.seg_len) {
      // past the end of the segment the last row was read, which may hold an infinity, and 0 * inf is NaN
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < ND; ++i)
          if (j0 + 4 * lg + v >= w.seg_len) vf[v][i] = 0.f;
    }
    f32v4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][e], q[i][e], s, 0, 0, 0);
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (j0 + 4 * lg + v >= w.seg_len) s[v] = -INFINITY;
      mx = fmaxf(mx, s[v]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_old = m;
    m = fmaxf(m, mx);
    // -inf as long as all scores are: such keys weigh nothing (exp(-inf - 0) = 0, not exp(-inf + inf))
    const float mn = m == -INFINITY ? 0.f : m;
    const float al = expf(m_old - mn);
    l *= al;
#pragma unroll
    for (int i = 0; i < ND; ++i) o[i] *= al;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float p = expf(s[v] - mn);
      l += p;
#pragma unroll
      for (int i = 0; i < ND; ++i) o[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v][i], p, o[i], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
#pragma unroll
  for (int i = 0; i < ND; ++i) *reinterpret_cast<f32v4*>(&so[wave][lr][16 * i + 4 * lg]) = o[i];
  if (lg == 0) { sm[wave][lr] = m; sl[wave][lr] = l; }
  __syncthreads();
  // waves that saw no key, or only scores of -inf, hold m = -inf, l = 0, o = 0: their weight is exp(-inf) = 0
  for (int e = tid; e < BQ * DH; e += 256) {
    const int r = e / DH, c = e - r * DH;
    if (r >= w.nq) break;
    const float mx = fmaxf(fmaxf(sm[0][r], sm[1][r]), fmaxf(sm[2][r], sm[3][r]));
    float den = 0.f, num = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f = expf(sm[i][r] - mx);
      den += f * sl[i][r];
      num += f * so[i][r][c];
    }
    reinterpret_cast<float*>(a.out)[(size_t)(w.q0 + r) * a.ldo + head * DH + c] = num / den;
  }
}

hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t s) {
  if (a.n_work == 0 || a.heads == 0) return hipSuccess;
  if (a.heads > 65535) return hipErrorInvalidValue;
  dim3 grid((unsigned)a.n_work, (unsigned)a.heads), block(256);
#define TCMV_ATTN32_CASE(D)                                                  \
  case D:                                                                    \
    hipLaunchKernelGGL((attn_f32_kernel<D>), grid, block, 0, s, a);          \
    break;
  switch (a.dh) {
    TCMV_ATTN32_CASE(16) TCMV_ATTN32_CASE(32) TCMV_ATTN32_CASE(48) TCMV_ATTN32_CASE(64)
    TCMV_ATTN32_CASE(80) TCMV_ATTN32_CASE(96) TCMV_ATTN32_CASE(112) TCMV_ATTN32_CASE(128)
    default: return hipErrorInvalidValue;
  }
#undef TCMV_ATTN32_CASE
  return hipGetLastError();
}

// hidden[cls_rows[i]][:] = cls + pos0[0]
__global__ void cls_rows_kernel(float* hidden, const int32_t* cls_rows, int n, const float* cls, const float* pos0,
                                int d) {
  const int i = blockIdx.x;
  float* dst = hidden + (size_t)cls_rows[i] * d;
  for (int c = threadIdx.x; c < d; c += blockDim.x) dst[c] = cls[c] + (pos0 ? pos0[c] : 0.f);
}

hipError_t launch_cls_rows(float* hidden, const int32_t* cls_rows, int n, const float* cls, const float* pos0, int d,
                           hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(cls_rows_kernel, dim3((unsigned)n), dim3(256), 0, s, hidden, cls_rows, n, cls, pos0, d);
  return hipGetLastError();
}

}  // namespace tcmv
