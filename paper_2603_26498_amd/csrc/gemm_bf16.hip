// C = epilogue(A * W^T + bias) on bf16 MFMA (gfx950), fp32 accumulation.
//
// A [m, k] and W [n, k] are both contiguous along k, so both operands are staged
// the same way: direct global -> LDS loads (16 bytes per lane, no registers in
// between) into tiles of 64 k-elements per row (128 bytes), with the 16-byte
// chunk index XOR-swizzled by (row/2)%8 so that the per-lane 16-byte MFMA operand
// reads are conflict-free.  LDS holds two to four such tiles and the loads of
// the next ones are in flight during the current tile's MFMAs.  Each wave owns a (BM/WM) x (BN/WN)
// sub-tile built from v_mfma_f32_32x32x16_bf16.
//
// The MFMA is issued with W as the row operand and A as the column operand, so
// the accumulator holds C^T: a lane owns ONE output row (token) and, per 32x32
// tile, four groups of four consecutive output columns.  Written out like that a
// store instruction would touch 32 rows; each wave therefore passes its sub-tile
// through a private LDS buffer (32 rows x 64 columns at a time) and comes back
// with lanes running along the row, 8 consecutive columns per lane: bias /
// position adds, GELU, the gated product, the rotary rotation, the fp32 residual
// read-modify-write and the stores all work on 16 or 32 contiguous bytes per
// lane.  All reads of a group (staged sums, old residual values) are issued
// before the first result is computed, so their round trips overlap instead of
// queueing behind each other.  Only the transposed-V columns of the QKV
// projection leave from registers (consecutive lanes = consecutive tokens = the
// contiguous direction of that buffer).
//
// Large products run on a PERSISTENT kernel: one workgroup of 8 waves per CU walks
// a list of 256x320 (or 256x256) tiles.  While it finishes the k-loop of one tile
// it already requests the first k-tile of its next tile, the tile is written out
// from the stage that is free by then, and the stores drain while the next
// k-loop runs.  Operands are read through buffer descriptors (base and size in
// SGPRs, one 32-bit lane offset per operand, everything else in the scalar
// offset), and the last tile of a dimension is shifted back to end at the matrix
// edge so that no load ever leaves the operand (its repeated rows / columns are
// skipped when it is written out).
// Smaller products use one workgroup per tile, from a set of tile shapes of which the launcher takes the one it
// estimates to be fastest (kTileKernels).  What bounds them is how long a k-tile takes to arrive (with two stages it is
// requested one iteration ahead) and the bytes that go from L2 to LDS (128x128 tiles: 11 TB/s at 700 TFLOP/s), so
// these kernels keep up to four stages in flight and the tiles that fill LDS once per CU may let two waves share a
// sub-tile, each with half of the k-steps: the wave tiles stay large (64x160: 7 fragment reads for 10 MFMAs) where the
// workgroup's is small.  With weights from memory, against two stages and 128x128 or 64x64 tiles only: 4096 x 1280 x 5120
// 79 -> 63 us; 256 x 3840 x 1280 18.4 -> 11.5; 64 x 5120 x 5120 57 -> 34.
// A long contraction over few rows that accumulates into the residual stream is cut into four slices of k whose
// fp32 partial sums a second kernel, or the norm that reads the stream next, adds in slice order.
//
// Workgroups are numbered so that the eight XCDs (workgroup id mod 8) each walk
// a contiguous range of tiles: neighbouring tiles share A rows or W rows in the
// XCD's own L2.
#include <algorithm>
#include <type_traits>
#include "tcmv_internal.h"
#include "device_utils.h"

namespace tcmv {

namespace {
typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;
constexpr int kEpStride = 68;                      // floats per row of a wave's staging buffer (64 columns + 4: conflict-free)
constexpr int kEpWaveBytes = 32 * kEpStride * 4;   // staging bytes per wave
}  // namespace

// Lane exchanges inside a row of 16 lanes through the data-parallel path of the vector ALU (no LDS round trip):
// value of lane (l ^ 1), lane (l ^ 2), lane (l + 4), lane (l + 8); lanes that would read past the row get 0.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_xor1(float v) { return dpp_move<0xB1>(v); }   // quad_perm [1,0,3,2]
__device__ __forceinline__ float lane_xor2(float v) { return dpp_move<0x4E>(v); }   // quad_perm [2,3,0,1]
__device__ __forceinline__ float lane_up4(float v) { return dpp_move<0x104>(v); }   // row_shl:4
__device__ __forceinline__ float lane_up8(float v) { return dpp_move<0x108>(v); }   // row_shl:8

// Rows and columns of the output that a workgroup may write: [row_lo, row_hi) x [col_lo, col_hi).
struct TileBounds { int64_t row_lo, row_hi; int col_lo, col_hi; int slice; };

// Writes one wave's sub-tile (MI x NI accumulator tiles of 32 x 32, first row m_base, first column wcol0).  In the
// accumulator a lane holds row (lane & 31) and columns 8*(v/4) + 4*(lane>>5) + v%4 of each tile.  The sub-tile
// leaves through the wave's private LDS buffer `ep` (32 rows x 64 columns of fp32 at a time) and comes back with
// lanes running along the rows, 8 consecutive columns per lane.  FULL: every element is inside the bounds.
//
// Key-norm maxima (EPI_QKV with g.kmax2, wave tiles of key columns that hold whole heads): on their way out the
// lanes square and sum their 8 values, the lanes of a row are added per head in a fixed order, and one lane per row
// accumulates the sums in the four spare floats at the end of the row's line in the staging buffer.  After the
// last column group of a 32-row block, the largest row of each segment goes to kmax2[segment][head] (the sums are
// >= 0, so their float bits order like unsigned integers).  The sums are taken before the rotary rotation (which
// preserves the norm of every pair) and before rounding to bf16 (which changes a squared norm by less than 2^-7 of
// itself): the factor 1.008 keeps the result an upper bound of the norm of the stored keys.
template <int EPI, int MI, int NI, bool FULL>
__device__ __forceinline__ void wave_epilogue(f32x16 (&acc)[MI][NI], const GemmArgs& g, float* ep, int64_t m_base, int wcol0,
                                              int lane, const TileBounds& tb) {
  constexpr int EPS = kEpStride;
  constexpr int TN = NI * 32;
  constexpr bool ROPE = EPI == EPI_QKV_ROPE, QKV = EPI == EPI_QKV || ROPE;
  const int lr = lane & 31, lg = lane >> 5;
  const bool kn = QKV && g.kmax2 != nullptr && wcol0 >= g.qcols && wcol0 < g.split;
  // heads are 64 or 80 columns wide where key norms are computed: divisions by constants (by a variable, three in every
  // column group: QKV of 4096 tokens 50.9 -> 50.0 us, of 16656 173.4 -> 170.5)
  auto head_of = [&](int col) { return g.kn_dh == 64 ? col / 64 : col / 80; };
  // old values of a group of the output (residual epilogues)
  auto load_old = [&](auto ngc, int nb, int64_t rbase, float4 (&o)[4][2]) {
    constexpr int NGT = decltype(ngc)::value;
    constexpr int LPR = NGT * 4, RPP = 64 / LPR, NP = 32 / RPP;
    const int col = wcol0 + nb * 32 + (lane % LPR) * 8;
    const int r0 = lane / LPR;
    const bool col_ok = FULL || (col >= tb.col_lo && col < tb.col_hi);
#pragma unroll
    for (int ps = 0; ps < NP; ++ps) {
      const int64_t row = rbase + ps * RPP + r0;
      if (FULL || (row >= tb.row_lo && row < tb.row_hi && col_ok)) {
        const float4* c = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(g.c) + (size_t)row * g.ldc + col);
        o[ps][0] = c[0]; o[ps][1] = c[1];
      }
    }
  };
  // `ahead` (EPI_RESID_AHEAD): old values of this group, requested while the previous group was written out;
  // `prefetch` requests those of the next group once this group's accumulators are in LDS and their registers free
  auto flush = [&](auto ngc, int mi, int nb, int64_t rbase, float4 (&ahead)[4][2], auto&& prefetch) {
    constexpr int NGT = decltype(ngc)::value;
    constexpr int LPR = NGT * 4;                   // lanes per row (8 columns each)
    constexpr int RPP = 64 / LPR;                  // rows per pass
    constexpr int NP = 32 / RPP;                   // passes
    const int c8 = (lane % LPR) * 8;
    const int col = wcol0 + nb * 32 + c8;
    const int r0 = lane / LPR;
    const bool col_ok = FULL || (col >= tb.col_lo && col < tb.col_hi);
    float4 here[4][2];
    if (EPI == EPI_RESID) load_old(ngc, nb, rbase, here);
    float4 (&o)[4][2] = EPI == EPI_RESID_AHEAD ? ahead : here;
#pragma unroll
    for (int ni = 0; ni < NGT; ++ni)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq)
        *reinterpret_cast<float4*>(ep + lr * EPS + ni * 32 + 8 * vq + 4 * lg) =
            make_float4(acc[mi][nb + ni][4 * vq], acc[mi][nb + ni][4 * vq + 1], acc[mi][nb + ni][4 * vq + 2], acc[mi][nb + ni][4 * vq + 3]);
    prefetch();
    float4 b0 = make_float4(0.f, 0.f, 0.f, 0.f), b1 = b0;
    if (EPI != EPI_PARTIAL && g.bias && col_ok) { b0 = *reinterpret_cast<const float4*>(g.bias + col); b1 = *reinterpret_cast<const float4*>(g.bias + col + 4); }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // plain stores read all staged values of the group first; the epilogues that keep other values in registers
    // (old residual values, rotary factors, key-norm sums) read them pass by pass
    constexpr bool BATCH = EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_GATED || EPI == EPI_PARTIAL;
    float4 v[NP][2];
    if (BATCH) {
#pragma unroll
      for (int ps = 0; ps < NP; ++ps) {
        const int r = ps * RPP + r0;
        v[ps][0] = *reinterpret_cast<const float4*>(ep + r * EPS + c8);
        v[ps][1] = *reinterpret_cast<const float4*>(ep + r * EPS + c8 + 4);
      }
    }
    if (QKV && kn) {
      // this group's share of the squared key norms: per row, the lanes of the first head of the group and the
      // lanes of the second (a group of 64 columns meets at most two heads of 64 or more columns)
      const int h_first = head_of(nb * 32);
      const bool second = head_of(nb * 32 + c8) != h_first;
#pragma unroll
      for (int ps = 0; ps < NP; ++ps) {
        const int r = ps * RPP + r0;
        const int64_t row = rbase + r;
        const bool ok = FULL || (row >= tb.row_lo && row < tb.row_hi && col_ok);
        const float4 va = *reinterpret_cast<const float4*>(ep + r * EPS + c8), vb = *reinterpret_cast<const float4*>(ep + r * EPS + c8 + 4);
        const float y[8] = {va.x + b0.x, va.y + b0.y, va.z + b0.z, va.w + b0.w, vb.x + b1.x, vb.y + b1.y, vb.z + b1.z, vb.w + b1.w};
        float sq = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) sq = fmaf(y[j], y[j], sq);
        if (!ok) sq = 0.f;
        float s0 = second ? 0.f : sq, s1 = second ? sq : 0.f;
        // sums over the LPR (4 or 8) lanes of a row, in a fixed order; valid in the first lane of the row
        s0 += lane_xor1(s0); s1 += lane_xor1(s1);
        s0 += lane_xor2(s0); s1 += lane_xor2(s1);
        if (LPR == 8) { s0 += lane_up4(s0); s1 += lane_up4(s1); }
        if (lane % LPR == 0) {
          float* acc2 = ep + r * EPS + 64 + h_first;
          acc2[0] += s0;
          if (head_of(nb * 32 + NGT * 32 - 1) != h_first) acc2[1] += s1;
        }
      }
    }
    // col modulo the head size, by its reciprocal (exact below 2^32 / rope_dh)
    const int rot_col = ROPE ? col - (int)__umulhi((uint32_t)col, g.rope_inv) * g.rope_dh : 0;
    float4 rot[2][2];
#pragma unroll
    for (int ps = 0; ps < NP; ++ps) {
      if (ROPE && ps % 2 == 0) {
        // rotary factors of two passes in one request: asked for pass by pass, each waited behind the stores of the pass
        // before (windowed encoder, 32768 tokens, QKV 315 -> 310 us; 21 k tokens, heads of 64, 192 -> 181).  All four
        // passes at once do not fit the registers of the 256x320 kernel (96 spilled).
        const float* f = g.rope + (size_t)__builtin_amdgcn_readfirstlane((int)rbase) * g.rope_dh;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int r = (ps + j) * RPP + r0;
          if (FULL || (rbase + r >= tb.row_lo && rbase + r < tb.row_hi)) {
            const float4* cs = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(f) + (uint32_t)((r * g.rope_dh + rot_col) * 4));
            rot[j][0] = cs[0]; rot[j][1] = cs[1];
          }
        }
      }
      const int64_t row = rbase + ps * RPP + r0;
      if (!FULL && (row < tb.row_lo || row >= tb.row_hi || !col_ok)) continue;
      if (!BATCH) {
        const int r = ps * RPP + r0;
        v[ps][0] = *reinterpret_cast<const float4*>(ep + r * EPS + c8);
        v[ps][1] = *reinterpret_cast<const float4*>(ep + r * EPS + c8 + 4);
      }
      float x[8] = {v[ps][0].x + b0.x, v[ps][0].y + b0.y, v[ps][0].z + b0.z, v[ps][0].w + b0.w,
                    v[ps][1].x + b1.x, v[ps][1].y + b1.y, v[ps][1].z + b1.z, v[ps][1].w + b1.w};
      if (EPI == EPI_GATED) {
        uint2 pk;
        const float gate[4] = {x[0], x[2], x[4], x[6]};
        float h[4];
        silu4(gate, h);
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] *= x[2 * j + 1];
        pk.x = pack_bf16x2(h[0], h[1]); pk.y = pack_bf16x2(h[2], h[3]);
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(g.c) + (size_t)row * g.ldc + (col >> 1)) = pk;
      } else if (EPI == EPI_STORE || EPI == EPI_GELU || QKV) {
        if (QKV && col >= g.split) continue;
        if (QKV && col < g.qcols) {
#pragma unroll
          for (int j = 0; j < 8; ++j) x[j] *= g.qscale;
        }
        if (ROPE) {
          const float4 c0 = rot[ps % 2][0], c1 = rot[ps % 2][1];
          const float a0 = x[0], a1 = x[1], a2 = x[2], a3 = x[3], a4 = x[4], a5 = x[5], a6 = x[6], a7 = x[7];
          x[0] = a0 * c0.x - a1 * c0.y; x[1] = a0 * c0.y + a1 * c0.x;
          x[2] = a2 * c0.z - a3 * c0.w; x[3] = a2 * c0.w + a3 * c0.z;
          x[4] = a4 * c1.x - a5 * c1.y; x[5] = a4 * c1.y + a5 * c1.x;
          x[6] = a6 * c1.z - a7 * c1.w; x[7] = a6 * c1.w + a7 * c1.z;
        }
        if (EPI == EPI_GELU) {
#pragma unroll
          for (int j = 0; j < 8; ++j) x[j] = gelu_bf16(x[j]);
        }
        uint4 pk;
        pk.x = pack_bf16x2(x[0], x[1]); pk.y = pack_bf16x2(x[2], x[3]); pk.z = pack_bf16x2(x[4], x[5]); pk.w = pack_bf16x2(x[6], x[7]);
        *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(g.c) + (size_t)row * g.ldc + col) = pk;
      } else if (EPI == EPI_PARTIAL) {
        float4* c = reinterpret_cast<float4*>(g.partial + ((size_t)tb.slice * g.m + row) * g.n + col);
        c[0] = make_float4(x[0], x[1], x[2], x[3]);
        c[1] = make_float4(x[4], x[5], x[6], x[7]);
      } else if (EPI == EPI_RESID || EPI == EPI_RESID_AHEAD) {
        float4* c = reinterpret_cast<float4*>(reinterpret_cast<float*>(g.c) + (size_t)row * g.ldc + col);
        c[0] = make_float4(o[ps][0].x + x[0], o[ps][0].y + x[1], o[ps][0].z + x[2], o[ps][0].w + x[3]);
        c[1] = make_float4(o[ps][1].x + x[4], o[ps][1].y + x[5], o[ps][1].z + x[6], o[ps][1].w + x[7]);
      } else if (EPI == EPI_EMBED) {
        const int pi = g.pos_idx ? g.pos_idx[row] : 0;
        if (g.pos_kind == 1) {
          const float4* p0 = reinterpret_cast<const float4*>(g.pos0 + (size_t)pi * g.n + col);
          const float4 pa = p0[0], pb = p0[1];
          x[0] += pa.x; x[1] += pa.y; x[2] += pa.z; x[3] += pa.w; x[4] += pb.x; x[5] += pb.y; x[6] += pb.z; x[7] += pb.w;
        } else if (g.pos_kind == 2) {
          const float4* p0 = reinterpret_cast<const float4*>(g.pos0 + (size_t)(pi & 0xFFFF) * g.n + col);
          const float4* p1 = reinterpret_cast<const float4*>(g.pos1 + (size_t)(pi >> 16) * g.n + col);
          const float4 pa = p0[0], pb = p0[1], qa = p1[0], qb = p1[1];
          x[0] += pa.x + qa.x; x[1] += pa.y + qa.y; x[2] += pa.z + qa.z; x[3] += pa.w + qa.w;
          x[4] += pb.x + qb.x; x[5] += pb.y + qb.y; x[6] += pb.z + qb.z; x[7] += pb.w + qb.w;
        }
        const int64_t dst = g.dst_row ? (int64_t)g.dst_row[row] : row;
        float4* c = reinterpret_cast<float4*>(reinterpret_cast<float*>(g.c) + (size_t)dst * g.ldc + col);
        c[0] = make_float4(x[0], x[1], x[2], x[3]);
        c[1] = make_float4(x[4], x[5], x[6], x[7]);
      }
    }
    asm volatile("" ::: "memory");
  };

  if constexpr (EPI == EPI_RESID_AHEAD) {
    // Outputs that do not stay cached between the kernels that update them (hundreds of megabytes of residual stream):
    // all groups of the wave tile in one sequence, the old values of group i+1 on their way while group i is written out.
    // It costs registers (two sets of old values; the compiler spills a few dozen), which is why outputs that do stay
    // cached keep the plain form: measured 14 % faster on fc2 at 100 k tokens (0.5 GB), 1 - 3 % slower at 32 k and 65 k
    // tokens (0.17 and 0.34 GB), hence the launcher's threshold of 0.4 GB.
    constexpr int G = NI / 2 + (NI & 1);           // groups per 32-row block: pairs of 32-column tiles, then a single one
    float4 oa[4][2], ob[4][2];
    load_old(std::integral_constant<int, (NI >= 2 ? 2 : 1)>{}, 0, m_base, oa);
    static_for<MI * G>([&](auto gc) {
      constexpr int gi = decltype(gc)::value;
      constexpr int mi = gi / G, k = gi % G, nb = 2 * k, NGT = (nb + 2 <= NI) ? 2 : 1;
      auto pre = [&]() {
        if constexpr (gi + 1 < MI * G) {
          constexpr int mi2 = (gi + 1) / G, k2 = (gi + 1) % G, nb2 = 2 * k2, NGT2 = (nb2 + 2 <= NI) ? 2 : 1;
          if constexpr (gi % 2 == 0) load_old(std::integral_constant<int, NGT2>{}, nb2, m_base + mi2 * 32, ob);
          else load_old(std::integral_constant<int, NGT2>{}, nb2, m_base + mi2 * 32, oa);
        }
      };
      if constexpr (gi % 2 == 0) flush(std::integral_constant<int, NGT>{}, mi, nb, m_base + mi * 32, oa, pre);
      else flush(std::integral_constant<int, NGT>{}, mi, nb, m_base + mi * 32, ob, pre);
    });
    return;
  }
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    const int64_t rbase = m_base + mi * 32;
    if (QKV && kn && lane < 32) *reinterpret_cast<float4*>(ep + lane * EPS + 64) = make_float4(0.f, 0.f, 0.f, 0.f);
    if (QKV && wcol0 + TN > g.split) {
      const int64_t row = rbase + lr;
      if (FULL || (row >= tb.row_lo && row < tb.row_hi)) {
        const int vc = g.vcol[row];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const int col = wcol0 + ni * 32 + 8 * vq + 4 * lg;
            if (col >= g.split && (FULL || (col >= tb.col_lo && col < tb.col_hi))) {
              float4 b4 = make_float4(0.f, 0.f, 0.f, 0.f);
              if (g.bias) b4 = *reinterpret_cast<const float4*>(g.bias + col);
              uint16_t* vt = reinterpret_cast<uint16_t*>(g.vt) + (size_t)(col - g.split) * g.ldvt + vc;
              vt[0] = f32_to_bf16(acc[mi][ni][4 * vq] + b4.x);
              vt[g.ldvt] = f32_to_bf16(acc[mi][ni][4 * vq + 1] + b4.y);
              vt[2 * g.ldvt] = f32_to_bf16(acc[mi][ni][4 * vq + 2] + b4.z);
              vt[3 * g.ldvt] = f32_to_bf16(acc[mi][ni][4 * vq + 3] + b4.w);
            }
          }
      }
      if (wcol0 >= g.split) continue;
    }
    {
      float4 none[4][2];
#pragma unroll
      for (int nb = 0; nb + 2 <= NI; nb += 2) flush(std::integral_constant<int, 2>{}, mi, nb, rbase, none, [] {});
      if (NI & 1) flush(std::integral_constant<int, 1>{}, mi, NI - 1, rbase, none, [] {});
    }
    if (QKV && kn) {
      // rows of this block -> table.  Lane l < 32 reads the sums of row l (up to four heads per wave tile).
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      const float4 sums = *reinterpret_cast<const float4*>(ep + lr * EPS + 64);
      const float hs[4] = {sums.x, sums.y, sums.z, sums.w};
      const int64_t row = rbase + lr;
      const bool row_ok = FULL || (row >= tb.row_lo && row < tb.row_hi);
      const int seg = row_ok ? g.row_seg[row] : -1;
      const int seg_a = __builtin_amdgcn_readlane(seg, 0), seg_b = __builtin_amdgcn_readlane(seg, 31);
      const bool one_segment = __all(row_ok) && seg_a == seg_b;        // rows are ordered by segment
      const int head0 = head_of(wcol0 - g.qcols);
      const int nh = head_of(TN);
      // all table words of the block are read before any is compared: one memory round trip per block, not one per head
      uint32_t bits[4] = {0u, 0u, 0u, 0u}, seen[4] = {0u, 0u, 0u, 0u};
      const bool writer = one_segment ? lane == 0 : (row_ok && lg == 0);
      uint32_t* word = g.kmax2 + ((size_t)(one_segment ? seg_a : (row_ok ? seg : 0)) * g.kn_heads + head0) * kKmaxStride;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        if (h < nh) {
          float vmax = hs[h] * 1.008f;
          if (one_segment) {
            // largest of the 32 rows (lanes 0..31): inside each row of 16 lanes, then lanes 0 and 16
            vmax = fmaxf(vmax, lane_xor1(vmax));
            vmax = fmaxf(vmax, lane_xor2(vmax));
            vmax = fmaxf(vmax, lane_up4(vmax));
            vmax = fmaxf(vmax, lane_up8(vmax));
            vmax = fmaxf(__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, vmax), 0)),
                         __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, vmax), 16)));
          }
          bits[h] = __float_as_uint(vmax);
          if (writer) seen[h] = __hip_atomic_load(word + h * kKmaxStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      // *p = max(*p, v).  Thousands of waves update the few words of one table: the atomic is only issued when the
      // word, as this wave has just seen it, is smaller (a stale view only costs an atomic that changes nothing),
      // which leaves a handful of atomics per word instead of one per wave queued behind each other.
#pragma unroll
      for (int h = 0; h < 4; ++h)
        if (h < nh && writer && seen[h] < bits[h]) atomicMax(word + h * kKmaxStride, bits[h]);
    }
  }
}


// Waits until at most N vector-memory loads of this wave are in flight and its LDS reads are back, then for the other
// waves of the workgroup.  One block, so that nothing moves in between, and not __syncthreads: before that barrier the
// compiler drained all loads in the prologue and in the last iterations.
template <int N>
__device__ __forceinline__ void wait_loads_and_waves() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory"); }

template <int BM, int BN, int WM, int WN, int KW, int NSTAGE, int MINB, int EPI>
__global__ __launch_bounds__(WM* WN* KW * 64, MINB) void gemm_bf16_kernel(GemmArgs g) {
  constexpr int BK = 64, TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32;
  constexpr int ROWB = BK * 2;                     // bytes per staged row
  constexpr int CPR = BK / 8;                      // 16-byte chunks per row
  constexpr int SW_SHIFT = 1;                      // rows that share a swizzle value (span 256 bytes = all banks)
  constexpr int RPL = 64 / CPR;                    // rows covered by one wave-wide load
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB, STAGE = A_BYTES + B_BYTES;

  const int tiles_n = (g.n + BN - 1) / BN;
  const int tiles_m = (int)((g.m + BM - 1) / BM);
  const int nslice = (EPI == EPI_PARTIAL) ? g.ksplit : 1;   // slices of k (neighbouring workgroups take the slices of a tile)
  const int total = tiles_m * tiles_n * nslice;
  const int chunk = (total + 7) >> 3;
  const int pq = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
  if (pq >= total) return;
  const int p = pq / nslice, slice = pq - p * nslice;
  // tiles are walked in groups of GM rows of tiles, column by column inside a group: the
  // workgroups that run at the same time on one XCD then form a roughly square block of
  // tiles and share both A rows and W rows in that XCD's L2
  constexpr int GM = 8;
  const int per_group = GM * tiles_n;
  const int grp = p / per_group, within = p - grp * per_group;
  const int gm_eff = min(GM, tiles_m - grp * GM);
  const int tn = within / gm_eff;
  const int tm = grp * GM + (within - tn * gm_eff);
  const int64_t m0 = (int64_t)tm * BM;
  const int n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN % WM, wn = wave % WN, kw = KW > 1 ? wave / (WM * WN) : 0;
  const uint16_t* A = reinterpret_cast<const uint16_t*>(g.a);
  const uint16_t* W = reinterpret_cast<const uint16_t*>(g.w);

  // Tile staging: global -> LDS directly.  One wave-wide load writes 64 consecutive
  // 16-byte chunks (RPL rows) of the stage; each lane fetches the global chunk that
  // belongs at its swizzled LDS position.  Rows past the end of the operand are
  // clamped to its last row (they only feed outputs that are never stored).
  constexpr int WAVES = WM * WN * KW;
  constexpr int NLA = BM / RPL / WAVES, NLB = BN / RPL / WAVES;      // wave-loads per wave and k-tile
  static_assert(BM % (RPL * WAVES) == 0 && BN % (RPL * WAVES) == 0, "tile/waves mismatch");
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  uint32_t offa[NLA], offb[NLB];
  {
    const int rl = lane / CPR, pc = lane % CPR;
#pragma unroll
    for (int i = 0; i < NLA; ++i) {
      const int row = (wave_u + WAVES * i) * RPL + rl;
      int64_t gr = m0 + row;
      if (gr > g.m - 1) gr = g.m - 1;
      offa[i] = (uint32_t)(gr * g.lda) + ((pc ^ ((row >> SW_SHIFT) & (CPR - 1))) << 3);
    }
#pragma unroll
    for (int i = 0; i < NLB; ++i) {
      const int row = (wave_u + WAVES * i) * RPL + rl;
      int gn = n0 + row;
      if (gn > g.n - 1) gn = g.n - 1;
      offb[i] = (uint32_t)gn * (uint32_t)g.k + ((pc ^ ((row >> SW_SHIFT) & (CPR - 1))) << 3);
    }
  }
  const int nk = g.k / BK / nslice;               // k-tiles of this workgroup
  const int k_first = slice * nk;
  auto load_tiles = [&](int kt, int buf) {
    uint8_t* sa = smem + buf * STAGE;
    uint8_t* sb = sa + A_BYTES;
    const uint16_t* ak = A + (size_t)(k_first + kt) * BK;
    const uint16_t* wk = W + (size_t)(k_first + kt) * BK;
#pragma unroll
    for (int i = 0; i < NLA; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(ak + offa[i]), (lptr_t)(sa + (wave_u + WAVES * i) * 1024), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < NLB; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(wk + offb[i]), (lptr_t)(sb + (wave_u + WAVES * i) * 1024), 16, 0, 0);
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;

  // NSTAGE LDS stages.  The barrier of a k-tile sits before its LAST k-step, not before its first: by then every
  // wave has read all of the tile's fragments into registers (so the tile's stage can be refilled with tile
  // kt+NSTAGE right after the barrier) and tile kt+1 has had at least three quarters of an iteration to land; only
  // its loads are waited for, those of the NSTAGE-2 tiles behind it stay in flight.  After the barrier a wave asks
  // for the first fragments of tile kt+1 and then still has the MFMAs of the last k-step of tile kt to issue, so no
  // wave sits behind a barrier with nothing to do while its fragments travel.
  static_assert(NSTAGE >= 2 && (NSTAGE - 1) * (NLA + NLB) <= 63, "loads in flight are counted in six bits");
  constexpr int KK = BK / 16 / KW;      // k-steps of a wave in a k-tile
  static_assert(KK % 2 == 0, "the register buffers alternate");
  const int lr = lane & 31, lg = lane >> 5;
  bf16x8 af[2][MI], bfr[2][NI];        // fragments double-buffered in registers
  auto frags = [&](int stage, int kk, int b) {
    const uint8_t* sa = smem + stage * STAGE;
    const uint8_t* sb = sa + A_BYTES;
    const int ch = (kw * KK + kk) * 2 + lg;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const int row = wm * TM + mi * 32 + lr;
      af[b][mi] = *reinterpret_cast<const bf16x8*>(sa + row * ROWB + ((ch ^ ((row >> SW_SHIFT) & (CPR - 1))) << 4));
    }
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int row = wn * TN + ni * 32 + lr;
      bfr[b][ni] = *reinterpret_cast<const bf16x8*>(sb + row * ROWB + ((ch ^ ((row >> SW_SHIFT) & (CPR - 1))) << 4));
    }
  };
  auto mfmas = [&](int b) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[b][ni], af[b][mi], acc[mi][ni], 0, 0, 0);
  };
  constexpr int NL = NLA + NLB;
#pragma unroll
  for (int i = 0; i < NSTAGE; ++i)
    if (i < nk) load_tiles(i, i);
  if (nk >= NSTAGE) wait_loads_and_waves<(NSTAGE - 1) * NL>();
  else wait_loads_and_waves<0>();
  // tile 0 is visible to all waves
  frags(0, 0, 0);
  // REST: k-tiles behind this one, NSTAGE standing for "at least NSTAGE" (tile kt+NSTAGE is then requested)
  auto iteration = [&](int kt, int cur, auto rest_c) {
    constexpr int REST = decltype(rest_c)::value;
    const int next = cur + 1 == NSTAGE ? 0 : cur + 1;
#pragma unroll
    for (int kk = 0; kk + 1 < KK; ++kk) {
      frags(cur, kk + 1, (kk + 1) & 1);
      mfmas(kk & 1);
      {
        // issue order of this k-step: one LDS read after each MFMA while reads are left, then the other MFMAs
        // (instead of all reads first): 2-5 % on the large products
        constexpr int NR = MI + NI, NM = MI * NI;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          if (i < NM) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if (NM > NR) __builtin_amdgcn_sched_group_barrier(0x008, NM - NR, 0);
      }
    }
    if (REST >= 1) {
      wait_loads_and_waves<(REST >= NSTAGE ? NSTAGE - 2 : REST - 1) * NL>();
      if (REST == NSTAGE) load_tiles(kt + NSTAGE, cur);
      frags(next, 0, 0);
    }
    mfmas((KK - 1) & 1);
    if (REST >= 1) {
      // after the barrier: an MFMA first, then the tile loads and fragment reads one by one between the MFMAs
      constexpr int NR = MI + NI, NM = MI * NI, NV = (REST == NSTAGE) ? NL : 0;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i < NV) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        if (i < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    }
  };
  {
    int kt = 0, cur = 0;
    auto step = [&] { ++kt; cur = cur + 1 == NSTAGE ? 0 : cur + 1; };
    for (; kt + NSTAGE < nk; step()) iteration(kt, cur, std::integral_constant<int, NSTAGE>{});
    static_for<NSTAGE>([&](auto i) {
      constexpr int rest = NSTAGE - 1 - decltype(i)::value;
      if (nk - 1 - kt >= rest) { iteration(kt, cur, std::integral_constant<int, rest>{}); step(); }
    });
  }

  // ---- epilogue: through the operand stages, which every wave has finished with
  static_assert(WAVES * kEpWaveBytes <= NSTAGE * STAGE, "epilogue staging does not fit in the operand stages");
  __syncthreads();
  const TileBounds tb{0, g.m, 0, g.n, slice};
  const int wcol0 = n0 + wn * TN;
  const bool full = m0 + BM <= g.m && n0 + BN <= g.n;
  float* ep = reinterpret_cast<float*>(smem + wave * kEpWaveBytes);
  if constexpr (KW == 1) {
    const int64_t m_base = m0 + wm * TM;
    if (full) wave_epilogue<EPI, MI, NI, true>(acc, g, ep, m_base, wcol0, lane, tb);
    else wave_epilogue<EPI, MI, NI, false>(acc, g, ep, m_base, wcol0, lane, tb);
  } else {
    // the two waves of a sub-tile hold the sums of different k-steps: each hands one half of its rows to the other
    static_assert(KW == 2 && MI % 2 == 0 && WAVES * (MI / 2) * NI * 4096 <= NSTAGE * STAGE, "exchange area");
    constexpr int H = MI / 2;
    f32x16 mine[H][NI];
    float4* out = reinterpret_cast<float4*>(smem) + (size_t)wave * H * NI * 256 + lane;
    const float4* in = reinterpret_cast<const float4*>(smem) + (size_t)(wave ^ (WM * WN)) * H * NI * 256 + lane;
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float t[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int v = 4 * q + j;
            t[j] = kw ? acc[h][ni][v] : acc[H + h][ni][v];
            mine[h][ni][v] = kw ? acc[H + h][ni][v] : acc[h][ni][v];
          }
          out[((h * NI + ni) * 4 + q) * 64] = make_float4(t[0], t[1], t[2], t[3]);
        }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 t = in[((h * NI + ni) * 4 + q) * 64];
          mine[h][ni][4 * q] += t.x; mine[h][ni][4 * q + 1] += t.y; mine[h][ni][4 * q + 2] += t.z; mine[h][ni][4 * q + 3] += t.w;
        }
    __syncthreads();
    const int64_t m_base = m0 + wm * TM + kw * (H * 32);
    if (full) wave_epilogue<EPI, H, NI, true>(mine, g, ep, m_base, wcol0, lane, tb);
    else wave_epilogue<EPI, H, NI, false>(mine, g, ep, m_base, wcol0, lane, tb);
  }
}

template <int BM, int BN, int WM, int WN, int KW, int NSTAGE, int MINB, bool SPLIT = false>
static hipError_t launch_cfg(const GemmArgs& a, hipStream_t s) {
  const int tiles_n = (a.n + BN - 1) / BN;
  const int64_t tiles_m = (a.m + BM - 1) / BM;
  const int64_t total = tiles_m * tiles_n * (a.epi == EPI_PARTIAL ? a.ksplit : 1);
  if (total <= 0) return hipSuccess;
  if (total > (1 << 30)) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)(((total + 7) / 8) * 8);
  const size_t lds = (size_t)NSTAGE * (BM + BN) * 128;
  dim3 block(WM * WN * KW * 64);
#define TCMV_GEMM_CASE(E)                                                                              \
  case E: {                                                                                            \
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, KW, NSTAGE, MINB, E>;                                 \
    if (lds > 64 * 1024) {                                                                             \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                          \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);        \
      if (e != hipSuccess) return e;                                                                   \
    }                                                                                                  \
    hipLaunchKernelGGL(kern, dim3(grid), block, lds, s, a);                                            \
    break;                                                                                             \
  }
  if constexpr (SPLIT) {
    switch (a.epi) {
      TCMV_GEMM_CASE(EPI_PARTIAL)
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (a.epi) {
      TCMV_GEMM_CASE(EPI_STORE) TCMV_GEMM_CASE(EPI_GELU) TCMV_GEMM_CASE(EPI_RESID)
      TCMV_GEMM_CASE(EPI_EMBED) TCMV_GEMM_CASE(EPI_QKV) TCMV_GEMM_CASE(EPI_QKV_ROPE) TCMV_GEMM_CASE(EPI_GATED)
      default: return hipErrorInvalidValue;
    }
  }
#undef TCMV_GEMM_CASE
  return hipGetLastError();
}

// C += bias + slice 0 + slice 1 + ... (in this order), 16 bytes per lane
__global__ __launch_bounds__(256) void splitk_reduce_kernel(float* c, int64_t ldc, const float* partial, const float* bias,
                                                            int64_t m, int n, int nslice) {
  const int n4 = n >> 2;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m * n4) return;
  const int64_t row = i / n4;
  const int col = (int)(i - row * n4) * 4;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (bias) acc = *reinterpret_cast<const float4*>(bias + col);
  for (int sl = 0; sl < nslice; ++sl) {
    const float4 v = *reinterpret_cast<const float4*>(partial + ((size_t)sl * m + row) * n + col);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  float4* dst = reinterpret_cast<float4*>(c + (size_t)row * ldc + col);
  float4 old = *dst;
  old.x += acc.x; old.y += acc.y; old.z += acc.z; old.w += acc.w;
  *dst = old;
}

// One wave-wide 16-byte-per-lane load global -> LDS through a buffer descriptor over `bytes` bytes at `base` (base,
// size and `soff` are wave-uniform and live in SGPRs; `voff` is the lane's byte offset).  Lane l writes 16 bytes
// at lds + 16 l.
__device__ __forceinline__ void buffer_load_lds16(const void* base, uint32_t bytes, void* lds, uint32_t voff, uint32_t soff) {
  const uint64_t v = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), 0,
                                                                      (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lptr_t)lds, 16, voff, soff, 0, 0);
}

template <int BM, int BN, int WM, int WN, int EPI>
__global__ __launch_bounds__(WM* WN * 64, 1) void gemm_bf16_persist_kernel(GemmArgs g) {
  constexpr int BK = 64, TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32;
  constexpr int ROWB = BK * 2, CPR = 8, RPL = 8, WAVES = WM * WN, KK = BK / 16;
  constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB, STAGE = A_BYTES + B_BYTES;
  constexpr int EP_WAVE = kEpWaveBytes, EP_BYTES = WAVES * EP_WAVE;
  constexpr int EXTRA = EP_BYTES > STAGE ? (EP_BYTES - STAGE + 255) / 256 * 256 : 0;
  constexpr int NLA = BM / RPL / WAVES, NLB = BN / RPL / WAVES;
  static_assert(BM % (RPL * WAVES) == 0 && BN % (RPL * WAVES) == 0, "tile/waves mismatch");
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];      // [stage 0][extra][stage 1]

  const int tiles_n = (g.n + BN - 1) / BN;
  const int tiles_m = (int)((g.m + BM - 1) / BM);
  const int total = tiles_m * tiles_n;
  const int chunk = (total + 7) >> 3;
  const int xcd = (int)(blockIdx.x & 7), slot = (int)(blockIdx.x >> 3), nslot = (int)(gridDim.x >> 3);
  int pq = xcd * chunk + slot;
  const int pq_end = min((xcd + 1) * chunk, total);
  if (pq >= pq_end) return;
  constexpr int GM = 8;
  auto tile_of = [&](int p, int& tm, int& tn) {
    const int per_group = GM * tiles_n;
    const int grp = p / per_group, within = p - grp * per_group;
    const int gm_eff = min(GM, tiles_m - grp * GM);
    tn = within / gm_eff;
    tm = grp * GM + (within - tn * gm_eff);
  };

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave_u / WN, wn = wave_u % WN;
  const uint16_t* A = reinterpret_cast<const uint16_t*>(g.a);
  const uint16_t* W = reinterpret_cast<const uint16_t*>(g.w);
  const int nk = g.k / BK;

  // sizes of the operands in bytes (below 2^32: checked by the launcher)
  const uint32_t bytes_a = (uint32_t)(((uint64_t)(g.m - 1) * (uint64_t)g.lda + (uint64_t)g.k) * 2ull);
  const uint32_t bytes_w = (uint32_t)((uint64_t)g.n * (uint64_t)g.k * 2ull);
  // Tile loads: lane l of a wave-wide load fetches 16 bytes of row l/8 of an 8-row slab; the slab's first row, the
  // k offset and the slab index go into the scalar offset of the instruction, so one VGPR per operand is enough.
  // The last tile of a dimension is shifted back to end at the matrix edge (its first rows / columns then repeat
  // the previous tile's and are skipped when the tile is written out), so every load stays inside the operand.
  const int rl = lane / CPR, pc = lane % CPR;
  const int swz = ((rl >> 1) + 4 * (wave_u & 1)) & 7;            // (row >> 1) & 7 for row = (wave + 8 i) * 8 + rl
  const uint32_t lane_a = (uint32_t)rl * (uint32_t)g.lda * 2u + ((pc ^ swz) << 4);
  const uint32_t lane_w = (uint32_t)rl * (uint32_t)g.k * 2u + ((pc ^ swz) << 4);
  uint32_t tile_a = 0, tile_w = 0;                               // byte offset of the tile's first row (scalars)
  int row_lo = 0, col_lo = 0;                                    // first row / column this tile owns
  int64_t m0 = 0; int n0 = 0;
  auto set_tile = [&](int tm_, int tn_) {
    row_lo = tm_ * BM; col_lo = tn_ * BN;
    m0 = min((int64_t)row_lo, g.m - BM); n0 = min(col_lo, g.n - BN);
    tile_a = (uint32_t)(m0 * g.lda) * 2u;
    tile_w = (uint32_t)n0 * (uint32_t)g.k * 2u;
  };
  auto stage_ptr = [&](int s) { return smem + (s ? STAGE + EXTRA : 0); };
  auto load_tiles = [&](int kt, int s, uint32_t ta, uint32_t tw) {
    uint8_t* sa = stage_ptr(s);
    uint8_t* sb = sa + A_BYTES;
    const uint32_t koff = (uint32_t)kt * (BK * 2);
    const uint32_t slab_a = (uint32_t)(8 * g.lda * 2), slab_w = (uint32_t)(8 * g.k * 2);
#pragma unroll
    for (int i = 0; i < NLA; ++i)
      buffer_load_lds16(A, bytes_a, sa + (wave_u + WAVES * i) * 1024, lane_a, ta + koff + (uint32_t)(wave_u + WAVES * i) * slab_a);
#pragma unroll
    for (int i = 0; i < NLB; ++i)
      buffer_load_lds16(W, bytes_w, sb + (wave_u + WAVES * i) * 1024, lane_w, tw + koff + (uint32_t)(wave_u + WAVES * i) * slab_w);
  };

  f32x16 acc[MI][NI];
  const int lr = lane & 31, lg = lane >> 5;
  bf16x8 af[2][MI], bfr[2][NI];
  auto frags = [&](int s, int kk, int b) {
    const uint8_t* sa = stage_ptr(s);
    const uint8_t* sb = sa + A_BYTES;
    const int ch = kk * 2 + lg;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const int row = wm * TM + mi * 32 + lr;
      af[b][mi] = *reinterpret_cast<const bf16x8*>(sa + row * ROWB + ((ch ^ ((row >> 1) & 7)) << 4));
    }
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int row = wn * TN + ni * 32 + lr;
      bfr[b][ni] = *reinterpret_cast<const bf16x8*>(sb + row * ROWB + ((ch ^ ((row >> 1) & 7)) << 4));
    }
  };
  auto mfmas = [&](int b) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[b][ni], af[b][mi], acc[mi][ni], 0, 0, 0);
  };

  {
    int tm, tn;
    tile_of(pq, tm, tn);
    set_tile(tm, tn);
  }
  int base = 0;                                  // stage of k-tile kt of the current tile = (kt + base) & 1
  load_tiles(0, 0, tile_a, tile_w);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (nk > 1) load_tiles(1, 1, tile_a, tile_w);
  frags(0, 0, 0);

  // MODE 2: after the barrier request k-tile kt+2 of this tile; 3: request k-tile 0 of the next tile (if there is one);
  // 0: last k-tile, nothing after it
  auto iteration = [&](int kt, auto mode_c, int np, bool has_next) {
    constexpr int MODE = decltype(mode_c)::value;
    const int cur = (kt + base) & 1;
#pragma unroll
    for (int kk = 0; kk + 1 < KK; ++kk) {
      frags(cur, kk + 1, (kk + 1) & 1);
      mfmas(kk & 1);
      {
        constexpr int NR = MI + NI, NM = MI * NI;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          if (i < NM) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if (NM > NR) __builtin_amdgcn_sched_group_barrier(0x008, NM - NR, 0);
      }
    }
    if (MODE >= 2) {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __syncthreads();
      if (MODE == 2) load_tiles(kt + 2, cur, tile_a, tile_w);
      if (MODE == 3 && has_next) {
        int tm2, tn2;
        tile_of(np, tm2, tn2);
        const int64_t m2 = min((int64_t)tm2 * BM, g.m - BM);
        const int n2 = min(tn2 * BN, g.n - BN);
        load_tiles(0, cur, (uint32_t)(m2 * g.lda) * 2u, (uint32_t)n2 * (uint32_t)g.k * 2u);
      }
      frags(cur ^ 1, 0, KK & 1);
    }
    mfmas((KK - 1) & 1);
    if (MODE == 2) {
      constexpr int NR = MI + NI, NM = MI * NI, NV = NLA + NLB;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i < NV) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        if (i < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    }
  };

  for (;;) {
    const int np = pq + nslot;
    const bool has_next = np < pq_end;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    {
      int kt = 0;
      for (; kt + 2 < nk; ++kt) iteration(kt, std::integral_constant<int, 2>{}, np, has_next);
      if (kt + 1 < nk) { iteration(kt, std::integral_constant<int, 3>{}, np, has_next); ++kt; }
      iteration(kt, std::integral_constant<int, 0>{}, np, has_next);
    }
    const int s_last = (nk - 1 + base) & 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                               // every wave is done with the last stage; the next tile's first k-tile has landed
    {
      float* ep = reinterpret_cast<float*>(smem + (s_last ? STAGE : 0) + wave_u * EP_WAVE);
      const int64_t m_base = m0 + wm * TM;
      const int wcol0 = n0 + wn * TN;
      // The epilogue reads its arguments (a dozen pointers and sizes that the k-loop never touches) from the kernel
      // argument segment again, through a pointer the compiler cannot trace back: kept live across the k-loop they
      // overflow the scalar registers and come back from scratch memory one dependent load at a time.
      const __attribute__((address_space(4))) GemmArgs* ge =
          (const __attribute__((address_space(4))) GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(ge) : : "memory");
      const GemmArgs& g2 = *(const GemmArgs*)ge;
      // likewise the lane number: the epilogue's per-lane offsets are the same for every tile, and the compiler
      // would compute them once before the first k-loop and carry them through it
      int lane_e = lane;
      asm volatile("" : "+v"(lane_e));
      const TileBounds tb{row_lo, g2.m, col_lo, g2.n, 0};
      if (m0 == row_lo && n0 == col_lo) wave_epilogue<EPI, MI, NI, true>(acc, g2, ep, m_base, wcol0, lane_e, tb);
      else wave_epilogue<EPI, MI, NI, false>(acc, g2, ep, m_base, wcol0, lane_e, tb);
    }
    if (!has_next) break;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();                               // the staging area is free again
    pq = np;
    {
      int tm, tn;
      tile_of(pq, tm, tn);
      set_tile(tm, tn);
    }
    base = (base + nk) & 1;
    if (nk > 1) load_tiles(1, (1 + base) & 1, tile_a, tile_w);
    frags(base & 1, 0, 0);
  }
}

template <int BM, int BN, int WM, int WN>
static hipError_t launch_persist(const GemmArgs& a, hipStream_t s) {
  const int tiles_n = (a.n + BN - 1) / BN;
  const int64_t tiles_m = (a.m + BM - 1) / BM;
  const int64_t total = tiles_m * tiles_n;
  if (total <= 0) return hipSuccess;
  if (total > (1 << 30)) return hipErrorInvalidValue;
  constexpr int STAGE = (BM + BN) * 128, EP_BYTES = WM * WN * kEpWaveBytes;
  constexpr int EXTRA = EP_BYTES > STAGE ? (EP_BYTES - STAGE + 255) / 256 * 256 : 0;
  const size_t lds = 2 * STAGE + EXTRA;
  const unsigned grid = (unsigned)std::min<int64_t>(256, (total + 7) / 8 * 8);
  dim3 block(WM * WN * 64);
#define TCMV_PGEMM_CASE(E)                                                                             \
  case E: {                                                                                            \
    auto kern = gemm_bf16_persist_kernel<BM, BN, WM, WN, E>;                                           \
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                            \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);          \
    if (e != hipSuccess) return e;                                                                     \
    hipLaunchKernelGGL(kern, dim3(grid), block, lds, s, a);                                            \
    break;                                                                                             \
  }
  switch (a.epi) {
    TCMV_PGEMM_CASE(EPI_STORE) TCMV_PGEMM_CASE(EPI_GELU) TCMV_PGEMM_CASE(EPI_RESID) TCMV_PGEMM_CASE(EPI_RESID_AHEAD)
    TCMV_PGEMM_CASE(EPI_EMBED) TCMV_PGEMM_CASE(EPI_QKV) TCMV_PGEMM_CASE(EPI_QKV_ROPE) TCMV_PGEMM_CASE(EPI_GATED)
    default: return hipErrorInvalidValue;
  }
#undef TCMV_PGEMM_CASE
  return hipGetLastError();
}


namespace {
enum GemmKernel { GK_INVALID, GK_P320, GK_P256, GK_T192x256, GK_T256x160, GK_T256x128, GK_T128x160, GK_T128K2, GK_T128, GK_T64, GK_SPLIT128, GK_SPLIT64, GK_COUNT };

// Tile kernels and what one workgroup's tile costs: `base` microseconds (first loads, write-out) plus `per_k` for every 64
// elements of k.  Those with shared = 0 fill a CU's LDS: they run in rounds of 256 tiles, and each round after the first
// costs `more` on top.  Of the shared ones two (T128) or three (T64) run on a CU; the cost of a k-tile grows with the tiles
// per CU from a floor, the memory latency (`more`).  Products that accumulate read and write four bytes per element:
// 12.4 us for a 256x256 tile on a CU of its own (all CUs write out together), 0.8 where other tiles compute meanwhile.
// Fitted to 1373 products of fewer than 400 tiles of 256x256: every layer product of five encoders at 64 .. 23184 rows,
// measured inside passes over 12 layers, whose weights come from memory (they exceed the last-level cache), and single
// products over weights that do too, with k from 128 to 8192 and at random row counts.  The kernel with the lowest estimate
// is on average 0.5 % slower than the fastest (more than 5 % on 47 products, more than 10 % on 9); the estimates themselves
// are off by 14 % r.m.s.  Small requests have since found their weights in the caches (the attention launch reads them, see
// touches_weights), so a product takes less than its estimate, 256 x 5120 x 1280 12.2 us instead of 16; the order of the kernels
// holds: of 172 products of 64 - 4032 rows, each measured on every kernel in passes that touch weights, another than the chosen
// one would shorten the pass by 0.12 % on average, by 2.1 % at most (1458 x 1152 x 4352, in slices), by more than 1 us a layer on 5.
struct TileKernel { GemmKernel kernel; int bm, bn, wave_n, shared; float base, per_k, more; };
constexpr TileKernel kTileKernels[] = {
    {GK_P320, 256, 320, 160, 0, 7.7f, 1.63f, 0.f},       {GK_P256, 256, 256, 64, 0, 3.7f, 1.54f, 3.2f},
    {GK_T192x256, 192, 256, 128, 0, 10.1f, 1.27f, 1.2f}, {GK_T256x160, 256, 160, 160, 0, 5.3f, 1.07f, 1.8f},
    {GK_T256x128, 256, 128, 64, 0, 4.3f, 0.81f, 5.2f},   {GK_T128x160, 128, 160, 160, 0, 8.2f, 0.59f, 0.f},
    {GK_T128K2, 128, 128, 64, 0, 4.5f, 0.47f, 1.6f},     {GK_T128, 128, 128, 64, 1, 3.3f, 0.56f, 0.76f},
    {GK_T64, 64, 64, 32, 1, 3.3f, 0.22f, 0.33f}};

float tile_cost(const TileKernel& t, int64_t m, int n, int k, int slices, bool accumulates) {
  const int64_t tiles = ((m + t.bm - 1) / t.bm) * ((n + t.bn - 1) / t.bn) * slices;
  const float per_cu = (float)((tiles + 255) / 256), nk = (float)(k / 64 / slices);
  const float out = accumulates ? (t.shared ? 0.8f : 12.4f) * (float)(t.bm * t.bn) / 65536.f : 0.f;
  return t.shared ? t.base + nk * std::max(t.more, t.per_k * per_cu) + per_cu * out
                  : per_cu * (t.base + nk * t.per_k + out) + (per_cu - 1.f) * t.more;
}

// a wave tile of `wave_n` columns computes key norms: whole heads, at most four, starting at head boundaries
bool wave_tile_holds_heads(int wave_n, int qcols, int dh) {
  return (dh == 64 || dh == 80) && wave_n % dh == 0 && wave_n / dh <= 4 && qcols % wave_n == 0;
}

bool is_persistent(GemmKernel k) { return k == GK_P320 || k == GK_P256; }
bool is_sliced(GemmKernel k) { return k == GK_SPLIT128 || k == GK_SPLIT64; }

// Which kernel computes rows [0, rows) of a product and which the rows behind them, and the widths of their wave tiles and tiles.
struct GemmPart { GemmKernel kernel = GK_INVALID; int wave_n = 0, block_n = 0; };
struct GemmRoute { GemmPart first, rest; int64_t rows = 0; bool valid() const { return first.kernel != GK_INVALID; } };

// what key norms add: a tile that cannot compute them pays for the separate pass over the keys (12 - 20 us), one that can
// for the sums in its write-out (1 - 14 us; they grow with the rows and more with the smaller tiles)
float norm_cost(const GemmArgs& a, const TileKernel& t, int64_t m) {
  if (a.epi != EPI_QKV || !a.kn_dh) return 0.f;
  if (!wave_tile_holds_heads(t.wave_n, a.qcols, a.kn_dh) || (is_persistent(t.kernel) && a.n % t.bn)) return 13.f + 2e-4f * (float)m;
  return is_persistent(t.kernel) ? 3.f + 2e-4f * (float)m : 1.f + 5e-4f * (float)m;
}

// Estimate for a persistent kernel over whole rounds of tiles, where tile_cost falls short (the chip clocks lower when every
// CU computes): microseconds a round, by k-tiles and by what the write-out does, and for the last, partly filled round.
// Products that accumulate are narrow (a model's width) and read more of A from memory for a tile: they have constants of
// their own, fitted to 2400 products of 3000 - 102000 rows (off by 6 and 8 % r.m.s.); those of the others are least squares
// over 396 products each of 2500 - 102000 rows, n 1024 - 8192, k 1024 - 5120, weights from memory (3.8 and 3.6 %).
struct RoundCost { float base, full_k, part_k, part_k_fill, resid, store, gelu, qkv, gated; };
constexpr RoundCost kRoundCosts[2][2] = {                          // 256x320, 256x256; accumulating, the others
    {{6.1f, 2.13f, 1.01f, 0.97f, 18.5f}, {5.2f, 1.97f, 1.05f, 0.97f, 0.f, 5.5f, 9.0f, 8.9f, 6.2f}},
    {{3.5f, 1.95f, 0.98f, 0.93f, 15.6f}, {4.7f, 1.60f, 0.83f, 0.77f, 0.f, 4.3f, 7.2f, 7.3f, 4.6f}}};

float rounds_cost(const GemmArgs& a, const TileKernel& t, int64_t m) {
  const RoundCost& c = kRoundCosts[t.kernel == GK_P320 ? 0 : 1][a.epi == EPI_RESID ? 0 : 1];
  const int64_t tiles = ((m + t.bm - 1) / t.bm) * ((a.n + t.bn - 1) / t.bn);
  const float full = (float)(tiles / 256), fill = (float)(tiles % 256) / 256.f, part = fill > 0.f ? 1.f : 0.f, nk = (float)(a.k / 64);
  const float out = a.epi == EPI_RESID ? c.resid : a.epi == EPI_QKV ? c.qkv : a.epi == EPI_GATED ? c.gated : a.epi == EPI_STORE ? c.store : c.gelu;
  return c.base + nk * (full * c.full_k + part * (c.part_k + fill * c.part_k_fill)) + (full + 0.7f * part) * out + norm_cost(a, t, m);
}

// the kernel with the lowest estimate for `m` rows
const TileKernel* cheapest_tile(const GemmArgs& a, int64_t m, bool can_persist, float* cost) {
  const TileKernel* best = nullptr;
  for (const TileKernel& t : kTileKernels) {
    if (is_persistent(t.kernel) && (!can_persist || m < 256)) continue;
    const float c = tile_cost(t, m, a.n, a.k, 1, a.epi == EPI_RESID) + norm_cost(a, t, m);
    if (!best || c < *cost) { best = &t; *cost = c; }
  }
  return best;
}

GemmPart part(const TileKernel& t) { return {t.kernel, t.wave_n, t.bn}; }

// four slices of k for `m` rows, taken if estimated below *cost; added by the norm that follows (`deferred`) or by a kernel
void consider_slices(const GemmArgs& a, int64_t m, bool deferred, float* cost, GemmPart* chosen) {
  if (a.epi != EPI_RESID || a.k < (deferred ? 1024 : 2048) || (a.k / 64) % 4) return;
  const float elements = 1e-6f * (float)m * (float)a.n;
  for (const TileKernel& t : kTileKernels) {
    if (!t.shared) continue;
    const float c = tile_cost(t, m, a.n, a.k, 4, false) + (deferred ? 0.f : 2.9f) + (t.kernel == GK_T64 ? 5.f : 4.5f) * elements;
    if (c < *cost) { *cost = c; chosen->kernel = t.kernel == GK_T64 ? GK_SPLIT64 : GK_SPLIT128; }
  }
}

GemmRoute choose_route(const GemmArgs& a) {
  GemmRoute r;
  if (a.k <= 0 || a.k % 64 || a.lda % 8 || a.n <= 0 || a.n % 8 || a.ldc % 4) return r;
  if (a.epi == EPI_QKV && (a.split % 8)) return r;
  if (a.epi == EPI_QKV && a.rope && (a.rope_dh % 8 || a.rope_dh <= 0)) return r;
  if (a.epi == EPI_GATED && (a.ldc % 4)) return r;
  // operand element offsets are kept in 32 bits
  if ((double)a.m * (double)a.lda >= 4294967296.0 || (double)a.n * (double)a.k >= 4294967296.0) return r;
  r.rows = a.m;
  // The persistent kernels shift their last tile back to the matrix edge and address their operands in bytes, 32 bits.
  const bool can_persist = a.k >= 128 && a.m >= 256 && a.n >= 320 && a.epi != EPI_PARTIAL &&
                           (double)a.m * (double)a.lda < 2147483648.0 && (double)a.n * (double)a.k < 2147483648.0;
  // Persistent 256-row tiles (8 waves, one workgroup per CU) from about one and a half rounds of them over the 256
  // CUs.  A tile 320 columns wide is taken where it needs no more tile area x rounds than a 256-wide one (hidden
  // sizes that are multiples of 320 but not of 256, such as 1280).
  const int64_t big_tiles = ((a.m + 255) / 256) * ((a.n + 255) / 256);
  float cost = 0.f;
  if (big_tiles >= 400 && can_persist) {
    auto area = [&](int64_t bm, int64_t bn) {
      const int64_t t = ((a.m + bm - 1) / bm) * ((a.n + bn - 1) / bn);
      return ((t + 255) / 256) * bm * bn;
    };
    const int64_t wide = area(256, 320), square = area(256, 256);
    // at the same area, the one whose wave tiles hold whole heads where key norms are wanted: the separate pass over the
    // keys takes 21 us at 25772 rows with heads of 64, the square tiles 10 - 15 more than the 184 of the wide ones
    const bool norms = a.epi == EPI_QKV && a.kn_dh && wide == square && a.n % 256 == 0 && wave_tile_holds_heads(64, a.qcols, a.kn_dh) &&
                       !wave_tile_holds_heads(160, a.qcols, a.kn_dh);
    const TileKernel& t = kTileKernels[wide <= square && !norms ? 0 : 1];
    r.first = part(t);
    cost = tile_cost(t, a.m, a.n, a.k, 1, a.epi == EPI_RESID) + norm_cost(a, t, a.m);
  } else {
    // Smaller products: a few rounds of tiles at most, so the round that is only partly filled decides.  The kernel with
    // the lowest estimate is taken (4096 x 1280 x 5120: 63 us with 128x160 tiles, 79 with 128x128; 4096 x 5120 x 1280:
    // 54 with one round of 256x320 tiles, 75 with 128x128; 256 x 5120 x 1280: 16 with 64x64, 19 - 45 with larger tiles).
    r.first = part(*cheapest_tile(a, a.m, can_persist, &cost));
    // A contraction over few rows that accumulates (out-projection and fc2 of one small request): a quarter of k per
    // workgroup, added to C in a fixed order by a second kernel or by the norm that follows (defer_reduce), where that is
    // estimated to win in spite of it.  What it costs, the slices written and read again, grows with the output: measured
    // with the longer norm, 256 x 1280 x 1280 7 us against 10 unsplit, 576 rows 9.5 / 9.7; 256 x 1280 x 5120 14 / 30, 1024
    // rows 30 (128x128 tiles) / 42, 1440 rows 33 / 41, 1760 rows 48 / 48.
    if (a.partial) consider_slices(a, a.m, a.defer_reduce, &cost, &r.first);
  }
  // Products with at least one whole round of large tiles: a last round that is nearly empty takes about half as long as a
  // full one, more than the rows in it take as a product of their own.  Both persistent kernels, whole or cut behind their
  // whole rounds, against what was chosen so far; cut where that is estimated to win by 1 % and 3 us.  16656 rows: fc2 (1280 x
  // 5120) 242 -> 212 us, with the 272 rows behind the round in slices of k 200; fc1 224 -> 210; 23501 x 1280 x 5120 352 -> 307.
  // Of 2065 products of 3000 - 102000 rows measured both ways the better one would gain 7.2 % on average; this rule gains 6.9 %
  // and loses more than 2 % on 19, 5.3 % at most.
  // Left as they are: products outside the rows, contractions and widths the estimate is fitted to (2907 x 8192 x 1024 would
  // lose 4 %, 70138 x 2048 x 2048 into an accumulated output 10 %), and accumulating products over a short contraction whose
  // rest is half a round or more (21910 x 1280 x 1280, 8854 rows behind one round: 94 us whole, 101 cut).
  const bool short_sums = a.epi == EPI_RESID && a.k < 3072;
  if (can_persist && a.m >= 3000 && a.k >= 1024 && !(a.epi == EPI_RESID && a.n >= 2048) && !is_sliced(r.first.kernel)) {
    float best = is_persistent(r.first.kernel) ? rounds_cost(a, kTileKernels[r.first.kernel - GK_P320], a.m) : cost;
    best *= 0.99f;
    const bool persistent = big_tiles >= 400;
    for (int i = 0; i < 2; ++i) {
      const TileKernel& t = kTileKernels[i];
      const int64_t tiles_n = (a.n + t.bn - 1) / t.bn, whole = (a.m / 256) * tiles_n / 256;   // whole rounds
      if (persistent && r.first.kernel != t.kernel && !a.kn_dh) {
        const float c = rounds_cost(a, t, a.m);
        if (c < best) { best = c; r.first = part(t); r.rows = a.m; }
      }
      const int64_t rows = whole * 256 / tiles_n * 256;
      if (rows <= 0 || rows >= a.m || (short_sums && (float)(a.m - rows) * (float)a.n > 0.48f * 256.f * (float)(t.bm * t.bn))) continue;
      float c_rest = 0.f;
      const TileKernel* rest = cheapest_tile(a, a.m - rows, true, &c_rest);
      if (is_persistent(rest->kernel)) c_rest = rounds_cost(a, *rest, a.m - rows);
      else if (a.epi == EPI_GELU || a.epi == EPI_QKV) c_rest *= rest->kernel == GK_T64 ? 1.f : 1.25f;    // what tile_cost leaves out
      GemmPart tail = part(*rest);
      if (a.rest_partial && 4 * (a.m - rows) * a.n <= a.rest_floats) consider_slices(a, a.m - rows, false, &c_rest, &tail);
      const float c = rounds_cost(a, t, rows) + c_rest + 3.f;
      if (c < best) { best = c; r.first = part(t); r.rest = tail; r.rows = rows; }
    }
  }
  return r;
}

bool computes_key_norms(const GemmPart& p, const GemmArgs& a) {
  // whole heads per wave tile, wave tiles that start at head boundaries, no shifted last tile
  return wave_tile_holds_heads(p.wave_n, a.qcols, a.kn_dh) && (!is_persistent(p.kernel) || a.n % p.block_n == 0);
}
bool computes_key_norms(const GemmRoute& r, const GemmArgs& a) {
  return r.valid() && computes_key_norms(r.first, a) && (r.rows == a.m || computes_key_norms(r.rest, a));
}
}  // namespace

bool gemm_bf16_can_fuse_key_norms(int64_t m, int n, int k, int qcols, int dh) {
  if (dh != 64 && dh != 80) return false;
  GemmArgs a{};
  a.m = m; a.n = n; a.k = k; a.lda = k; a.ldc = 2 * qcols; a.epi = EPI_QKV; a.split = 2 * qcols; a.qcols = qcols; a.kn_dh = dh;
  return computes_key_norms(choose_route(a), a);
}

const char* gemm_bf16_kernel_name(const GemmArgs& a) {
  // GemmKernel order; then whole rounds of either persistent kernel followed by another for the rest
#define TCMV_NAMES(first) {first "256x320 persistent", first "256x256 persistent", first "192x256", first "256x160", first "256x128", \
                           first "128x160", first "128x128 k/2", first "128x128", first "64x64", first "128x128 slices", first "64x64 slices"}
  static const char* const names[3][GK_COUNT - 1] = {TCMV_NAMES(""), TCMV_NAMES("256x320 persistent + "), TCMV_NAMES("256x256 persistent + ")};
#undef TCMV_NAMES
  const GemmRoute r = choose_route(a);
  if (!r.valid()) return nullptr;
  return r.rows == a.m ? names[0][r.first.kernel - 1] : names[r.first.kernel == GK_P320 ? 1 : 2][r.rest.kernel - 1];
}

int gemm_bf16_slices(const GemmArgs& a) { return is_sliced(choose_route(a).first.kernel) ? 4 : 1; }

static hipError_t launch_part(GemmKernel gk, const GemmArgs& args, hipStream_t s) {
  GemmArgs a = args;
  // a kernel of its own: with the rotation the others keep fewer values in registers (QKV of 4096 tokens 52.3 -> 51.0 us)
  if (a.epi == EPI_QKV && a.rope) {
    a.epi = EPI_QKV_ROPE;
    a.rope_inv = 0xFFFFFFFFu / (uint32_t)a.rope_dh + 1;
  }
  if (is_persistent(gk) && a.epi == EPI_RESID && (double)a.m * (double)a.n * 4.0 > 400e6) {
    // An output larger than the last-level cache: see wave_epilogue.  By the rows of this part: heads of 377 MB before a rest
    // that takes the output above 400 lose by it (87000 - 91000 x 1152 x 1280 363 -> 376 us, k 4352 866 -> 879).
    GemmArgs g = a;
    g.epi = EPI_RESID_AHEAD;
    return gk == GK_P320 ? launch_persist<256, 320, 4, 2>(g, s) : launch_persist<256, 256, 2, 4>(g, s);
  }
  switch (gk) {
    case GK_P320: return launch_persist<256, 320, 4, 2>(a, s);
    case GK_P256: return launch_persist<256, 256, 2, 4>(a, s);
    case GK_SPLIT128:
    case GK_SPLIT64: {
      GemmArgs g = a;
      g.epi = EPI_PARTIAL; g.ksplit = 4;
      const hipError_t e = gk == GK_SPLIT64 ? launch_cfg<64, 64, 2, 2, 1, 3, 3, true>(g, s) : launch_cfg<128, 128, 2, 2, 1, 2, 2, true>(g, s);
      if (e != hipSuccess || a.defer_reduce) return e;
      const int64_t n4 = (int64_t)a.m * (a.n / 4);
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s,
                         reinterpret_cast<float*>(a.c), a.ldc, a.partial, a.bias, a.m, a.n, 4);
      return hipGetLastError();
    }
    case GK_T192x256: return launch_cfg<192, 256, 2, 2, 1, 2, 1>(a, s);
    case GK_T256x160: return launch_cfg<256, 160, 4, 1, 1, 3, 1>(a, s);
    case GK_T256x128: return launch_cfg<256, 128, 4, 2, 1, 3, 1>(a, s);
    case GK_T128x160: return launch_cfg<128, 160, 2, 1, 2, 4, 1>(a, s);
    case GK_T128K2: return launch_cfg<128, 128, 2, 2, 2, 4, 1>(a, s);
    case GK_T128: return launch_cfg<128, 128, 2, 2, 1, 2, 2>(a, s);
    case GK_T64: return launch_cfg<64, 64, 2, 2, 1, 3, 3>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// the product of rows [r0, m): every operand and output that has a row per row of A
static GemmArgs rows_from(const GemmArgs& a, int64_t r0) {
  GemmArgs g = a;
  const bool f32_out = a.epi == EPI_RESID || a.epi == EPI_EMBED;
  g.m = a.m - r0;
  g.a = reinterpret_cast<const uint16_t*>(a.a) + r0 * a.lda;
  if (!(a.epi == EPI_EMBED && a.dst_row)) g.c = reinterpret_cast<uint8_t*>(a.c) + r0 * a.ldc * (f32_out ? 4 : 2);
  if (a.dst_row) g.dst_row = a.dst_row + r0;
  if (a.pos_idx) g.pos_idx = a.pos_idx + r0;
  if (a.vcol) g.vcol = a.vcol + r0;
  if (a.rope) g.rope = a.rope + r0 * a.rope_dh;
  if (a.row_seg) g.row_seg = a.row_seg + r0;
  g.partial = a.rest_partial;
  g.defer_reduce = 0;
  return g;
}

hipError_t launch_gemm_bf16(const GemmArgs& a, hipStream_t s) {
  if (a.m == 0 || a.n == 0) return hipSuccess;
  const GemmRoute r = choose_route(a);
  if (a.epi == EPI_QKV && a.kmax2 && !(computes_key_norms(r, a) && a.split == 2 * a.qcols && a.row_seg)) return hipErrorInvalidValue;
  if (!r.valid()) return hipErrorInvalidValue;
  if (r.rows == a.m) return launch_part(r.first.kernel, a, s);
  GemmArgs head = a;
  head.m = r.rows;
  const hipError_t e = launch_part(r.first.kernel, head, s);
  return e != hipSuccess ? e : launch_part(r.rest.kernel, rows_from(a, r.rows), s);
}

}  // namespace tcmv
