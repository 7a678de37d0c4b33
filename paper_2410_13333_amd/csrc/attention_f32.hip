// fp32 causal attention of the all-fp32 validation mode, on v_mfma_f32_32x32x2_f32 (full fp32 products and sums): forward
// with online softmax; dQ (which also forms delta = dO . O of its rows); dK and dV.  No atomics: every sum has a fixed
// order.
//
// The kernels follow the bf16 ones: every score-like product is computed transposed, so that the softmax row is the
// result's lane column and the probabilities of a lane are the B operand of the next product as they stand: element
// 4g + r of a 32x32 result is row 8g + 4 (lane / 32) + r, and an MFMA that takes it as its B operand contracts over the
// two rows 8g + r and 8g + 4 + r, for which the A operand is read from memory as two 128-byte row pieces.  The products
// over the head dimension take 16 bytes per lane of either operand in the same manner (features 8G + 4 (lane / 32) ..
// +3).  Nothing passes through LDS on the way in.
//
// The shapes of this mode are small (a few heads, a few hundred positions), so the bound is the chain of blocks a
// wavefront walks, not the rate: a workgroup owns 32 rows, its four wavefronts take every fourth block of the other
// sequence index, and their partial results meet in a fixed tree through LDS.
// Measured (2 x 256 positions, 8 / 4 heads of 64): forward 3415 -> 13 us, dQ 4313 -> 17 us, dK and dV 13468 -> 38 us
// against the kernels this replaced (one thread per row, scalar loops); dQ, dK and dV in one launch, every query head's share of dK and dV
// in a workgroup of its own: 56 -> 30 us.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace {

// Template argument DT: 32-column tiles of a head vector (head_dim d = 16 .. 128 in steps of 16; features at or beyond d
// read as zero and are not stored).

// 16 bytes per feature group: element 4G + j is feature 8G + 4 hf + j of `row` (null: zeros)
template <int DT>
__device__ __forceinline__ void load_row(const float* row, int d, int hf, float (&f)[DT * 16]) {
#pragma unroll
  for (int G = 0; G < DT * 4; G++) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row && 8 * G < d) v = *reinterpret_cast<const float4*>(row + 8 * G + 4 * hf);
    f[4 * G] = v.x; f[4 * G + 1] = v.y; f[4 * G + 2] = v.z; f[4 * G + 3] = v.w;
  }
}
// A operand of a product that contracts over rows r0 .. r0+31 of m: element [e][t] is feature 32 t + lane % 32 of row
// r0 + 8 (e / 4) + 4 hf + e % 4; rows at or beyond `rows` read as zero
template <int DT>
__device__ __forceinline__ void load_cols(const float* __restrict__ m, int64_t ld, int r0, int rows, int d, int l32, int hf,
                                          float (&f)[16][DT]) {
#pragma unroll
  for (int e = 0; e < 16; e++) {
    const int r = r0 + 8 * (e >> 2) + 4 * hf + (e & 3);
#pragma unroll
    for (int t = 0; t < DT; t++) f[e][t] = r < rows && 32 * t + l32 < d ? m[int64_t(r) * ld + 32 * t + l32] : 0.f;
  }
}
template <int N>
__device__ __forceinline__ f32x16 dot_rows(const float (&a)[N], const float (&b)[N]) {
  f32x16 c;
#pragma unroll
  for (int e = 0; e < 16; e++) c[e] = 0.f;
#pragma unroll
  for (int q = 0; q < N; q++) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], c, 0, 0, 0);
  return c;
}
template <int DT>
__device__ __forceinline__ void accumulate(f32x16 (&acc)[DT], const float (&a)[16][DT], const f32x16& b) {
#pragma unroll
  for (int e = 0; e < 16; e++)
#pragma unroll
    for (int t = 0; t < DT; t++) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e][t], b[e], acc[t], 0, 0, 0);
}
// accumulate() for a block that the diagonal crosses.  There b holds zeros for the masked pairs, which take nothing from a
// finite row, but a row of `m` with an infinity or a NaN in it must not reach the positions that may not see it: then the
// sum is formed pair by pair over the allowed ones (allowed(r): row r counts for this lane's position).  sp: 32 x 32 floats
// of LDS of this wavefront.
template <int DT, class Allowed>
__device__ __forceinline__ void accumulate_diagonal(f32x16 (&acc)[DT], const float (&a)[16][DT], const f32x16& b,
                                                    const float* __restrict__ m, int64_t ld, int r0, int rows, int d, int l32,
                                                    int hf, float (*sp)[32], Allowed&& allowed) {
  float bad = 0.f;  // 0 * infinity and 0 * NaN are NaN
#pragma unroll
  for (int e = 0; e < 16; e++)
#pragma unroll
    for (int t = 0; t < DT; t++) bad += a[e][t] * 0.f;
  if (!__any(bad != bad)) {
    accumulate<DT>(acc, a, b);
    return;
  }
  auto sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  sync();
#pragma unroll
  for (int e = 0; e < 16; e++) sp[8 * (e >> 2) + 4 * hf + (e & 3)][l32] = b[e];
  sync();
#pragma unroll 1
  for (int r = 0; r < 32 && r0 + r < rows; r++) {
    if (!allowed(r0 + r)) continue;
    const float w = sp[r][l32];
#pragma unroll
    for (int t = 0; t < DT; t++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int f = 32 * t + 8 * g + 4 * hf;
        if (f < d)
#pragma unroll
          for (int j = 0; j < 4; j++) acc[t][4 * g + j] += w * m[int64_t(r0 + r) * ld + f + j];
      }
  }
  sync();
}
// sum of the four wavefronts' accumulators in wavefront 0: (0 + 2) + (1 + 3)
template <int DT>
__device__ __forceinline__ void sum_waves(f32x16 (&acc)[DT], float (*part)[DT * 16][64], int wave, int lane) {
#pragma unroll
  for (int half = 2; half > 0; half >>= 1) {
    __syncthreads();
    if (wave >= half && wave < 2 * half)
#pragma unroll
      for (int t = 0; t < DT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) part[wave - half][t * 16 + e][lane] = acc[t][e];
    __syncthreads();
    if (wave < half)
#pragma unroll
      for (int t = 0; t < DT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[t][e] += part[wave][t * 16 + e][lane];
  }
}
// Rotary tables; with them the backward turns dQ and dK back by the angle of their position as it stores them (cos null: not at all).
struct Unrotate {
  const float *cos_tab, *sin_tab;  // [S][d / 2]
};
// store a transposed result (lane column = row `row` of the output): four consecutive features per group
template <int DT>
__device__ __forceinline__ void store_row(float* row, const f32x16 (&acc)[DT], float mul, int d, int hf) {
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int f = 32 * t + 8 * g + 4 * hf;
      if (f < d)
        *reinterpret_cast<float4*>(row + f) =
            make_float4(acc[t][4 * g] * mul, acc[t][4 * g + 1] * mul, acc[t][4 * g + 2] * mul, acc[t][4 * g + 3] * mul);
    }
}
// the same turned back: the two halves of H groups of eight features each; group G is registers 4 (G % 4) .. of tile G / 4.  Straight to
// memory: turned back in place, for either head width of DT = 3, the compiler kept accumulators in scratch memory (192 bytes a lane), and the loops
// before lost (heads of 80, 681 positions, 25 heads: dQ 71.6 -> 83.5 us, dK and dV 111 -> 117).
template <int H, int DT>
__device__ __forceinline__ void store_row_halves(float* row, const f32x16 (&acc)[DT], float mul, const float* cs, const float* sn, int hf) {
#pragma unroll
  for (int g = 0; g < H; g++) {
    const float4 c = *reinterpret_cast<const float4*>(cs + 8 * g + 4 * hf), n = *reinterpret_cast<const float4*>(sn + 8 * g + 4 * hf);
    const float cv[4] = {c.x, c.y, c.z, c.w}, nv[4] = {n.x, n.y, n.z, n.w};
    float a[4], b[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float x = acc[g / 4][4 * (g % 4) + e] * mul, y = acc[(g + H) / 4][4 * ((g + H) % 4) + e] * mul;
      a[e] = x * cv[e] + y * nv[e];
      b[e] = y * cv[e] - x * nv[e];
    }
    *reinterpret_cast<float4*>(row + 8 * g + 4 * hf) = make_float4(a[0], a[1], a[2], a[3]);
    *reinterpret_cast<float4*>(row + 8 * (g + H) + 4 * hf) = make_float4(b[0], b[1], b[2], b[3]);
  }
}
// d is 32 DT or 16 less
template <int DT>
__device__ __forceinline__ void store_row(float* row, const f32x16 (&acc)[DT], float mul, const Unrotate& un, int pos, int d, int hf) {
  const float *cs = un.cos_tab + int64_t(pos) * (d >> 1), *sn = un.sin_tab + int64_t(pos) * (d >> 1);
  if (!un.cos_tab) store_row<DT>(row, acc, mul, d, hf);
  else if (d == 32 * DT) store_row_halves<2 * DT, DT>(row, acc, mul, cs, sn, hf);
  else store_row_halves<2 * DT - 1, DT>(row, acc, mul, cs, sn, hf);
}
template <int DT>
__device__ __forceinline__ void clear(f32x16 (&acc)[DT]) {
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int e = 0; e < 16; e++) acc[t][e] = 0.f;
}

// one-dimensional grid: query blocks of 32 (longest rows first), then batch rows, then heads
template <int DT>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(const float* __restrict__ qkv, int64_t ld, float* __restrict__ o,
                                                           int64_t ldo, float* __restrict__ lse, int b, int S, int nq, int nkv, int d) {
  __shared__ float part[2][DT * 16][64];
  __shared__ float sm[4][32], sl[4][32], sp[4][32][32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5;
  const int hq = blockIdx.x % nq, bi = blockIdx.x / nq % b, q0 = ((S + 31) / 32 - 1 - blockIdx.x / nq / b) * 32, hk = hq / (nq / nkv);
  const float* base = qkv + int64_t(bi) * S * ld;
  const float *K = base + int64_t(nq + hk) * d, *V = base + int64_t(nq + nkv + hk) * d;
  const int qi = q0 + l32;
  const float sc = rsqrtf((float)d);
  float q[DT * 16];
  load_row<DT>(qi < S ? base + int64_t(qi) * ld + int64_t(hq) * d : nullptr, d, hf, q);
  f32x16 acc[DT];
  clear(acc);
  float m = -INFINITY, l = 0.f;
  for (int j0 = wave * 32; j0 <= q0; j0 += 128) {
    float k[DT * 16], v[16][DT];
    load_row<DT>(j0 + l32 < S ? K + int64_t(j0 + l32) * ld : nullptr, d, hf, k);
    load_cols<DT>(V, ld, j0, S, d, l32, hf, v);
    f32x16 s = dot_rows(k, q);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int j = j0 + 8 * (e >> 2) + 4 * hf + (e & 3);
      s[e] = j <= qi ? s[e] * sc : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    const float mn = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, 64)));  // finite: j0 <= q0 <= qi
    const float corr = __expf(m - mn);
    l *= corr;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      s[e] = __expf(s[e] - mn);
      l += s[e];
    }
#pragma unroll
    for (int t = 0; t < DT; t++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[t][e] *= corr;
    m = mn;
    if (j0 < q0) accumulate<DT>(acc, v, s);
    else accumulate_diagonal<DT>(acc, v, s, V, ld, j0, S, d, l32, hf, sp[wave], [&](int j) { return j <= qi; });
  }
  // merge the four partial softmaxes: wavefront 0 always holds block 0, so the overall maximum is finite
  l += __shfl_xor(l, 32, 64);
  if (hf == 0) {
    sm[wave][l32] = m;
    sl[wave][l32] = l;
  }
  __syncthreads();
  const float M = fmaxf(fmaxf(sm[0][l32], sm[1][l32]), fmaxf(sm[2][l32], sm[3][l32]));
  const float w = __expf(m - M);
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int e = 0; e < 16; e++) acc[t][e] *= w;
  float L = 0.f;
#pragma unroll
  for (int i = 0; i < 4; i++) L += sl[i][l32] * __expf(sm[i][l32] - M);
  sum_waves<DT>(acc, part, wave, lane);
  if (wave != 0 || qi >= S) return;
  store_row<DT>(o + (int64_t(bi) * S + qi) * ldo + int64_t(hq) * d, acc, 1.f / L, d, hf);
  if (hf == 0) lse[(int64_t(bi) * nq + hq) * S + qi] = M + __logf(L);
}

// ---- backward: dQ, dK and dV.  TOGETHER: in one launch, where both parts form delta = dO . O of the rows they need; apart the dQ kernel
// forms it and the dK / dV kernel reads it.
// LDS of a workgroup: sums of wavefronts, and blocks on the diagonal
template <int DT>
struct BwdLds {
  float part[2][DT * 16][64], sp[4][32][32];
};
// dQ of query rows q0 .. q0 + 31
template <int DT, bool TOGETHER>
__device__ __forceinline__ void dq_block(BwdLds<DT>& lds, int q0, int hq, int bi, const float* __restrict__ qkv, int64_t ld, const float* __restrict__ o,
                                         int64_t ldo, const float* __restrict__ lse, const float* __restrict__ d_o, int64_t ldd,
                                         float* __restrict__ delta, float* __restrict__ dqkv, int64_t ldg, int S, int nq, int nkv, int d, Unrotate un) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5, hk = hq / (nq / nkv);
  const float* base = qkv + int64_t(bi) * S * ld;
  const float *K = base + int64_t(nq + hk) * d, *V = base + int64_t(nq + nkv + hk) * d;
  const int qi = q0 + l32;
  const bool live = qi < S;
  const float sc = rsqrtf((float)d);
  float q[DT * 16], dO[DT * 16];
  float dl = 0.f;
  load_row<DT>(live ? d_o + (int64_t(bi) * S + qi) * ldd + int64_t(hq) * d : nullptr, d, hf, dO);
  load_row<DT>(live ? o + (int64_t(bi) * S + qi) * ldo + int64_t(hq) * d : nullptr, d, hf, q);
#pragma unroll
  for (int i = 0; i < DT * 16; i++) dl += q[i] * dO[i];
  dl += __shfl_xor(dl, 32, 64);
  const int64_t si = (int64_t(bi) * nq + hq) * S + qi;
  if (!TOGETHER && wave == 0 && hf == 0 && live) delta[si] = dl;
  const float L = live ? lse[si] : 0.f;
  load_row<DT>(live ? base + int64_t(qi) * ld + int64_t(hq) * d : nullptr, d, hf, q);
  f32x16 acc[DT];
  clear(acc);
  for (int j0 = wave * 32; j0 <= q0; j0 += 128) {
    float k[DT * 16], kc[16][DT];
    load_row<DT>(j0 + l32 < S ? V + int64_t(j0 + l32) * ld : nullptr, d, hf, k);
    f32x16 dp = dot_rows(k, dO);
    load_row<DT>(j0 + l32 < S ? K + int64_t(j0 + l32) * ld : nullptr, d, hf, k);
    load_cols<DT>(K, ld, j0, S, d, l32, hf, kc);
    f32x16 s = dot_rows(k, q);
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int j = j0 + 8 * (e >> 2) + 4 * hf + (e & 3);
      s[e] = j <= qi ? __expf(s[e] * sc - L) * (dp[e] - dl) : 0.f;
    }
    if (j0 < q0) accumulate<DT>(acc, kc, s);
    else accumulate_diagonal<DT>(acc, kc, s, K, ld, j0, S, d, l32, hf, lds.sp[wave], [&](int j) { return j <= qi; });
  }
  sum_waves<DT>(acc, lds.part, wave, lane);
  if (wave != 0 || !live) return;
  store_row<DT>(dqkv + (int64_t(bi) * S + qi) * ldg + int64_t(hq) * d, acc, sc, un, qi, d, hf);
}

// dK and dV of key rows j0 .. j0 + 31 from the query heads hq0 .. hq0 + heads - 1 of their group: the wavefronts share out the (head, query
// block at or below the diagonal) pairs.  part: the sums go there, [dK | dV][b][n_q][S][d], at hq0.
template <int DT, bool TOGETHER>
__device__ __forceinline__ void dkv_block(BwdLds<DT>& lds, int j0, int hq0, int heads, int bi, int nb_all, const float* __restrict__ qkv, int64_t ld,
                                          const float* __restrict__ o, int64_t ldo, const float* __restrict__ lse, const float* __restrict__ d_o,
                                          int64_t ldd, const float* __restrict__ delta, float* __restrict__ dqkv, int64_t ldg, int S, int nq,
                                          int nkv, int d, float* __restrict__ part, Unrotate un) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5, hk = hq0 / (nq / nkv);
  const float* base = qkv + int64_t(bi) * S * ld;
  const int ji = j0 + l32;
  const float sc = rsqrtf((float)d);
  float k[DT * 16], v[DT * 16];
  load_row<DT>(ji < S ? base + int64_t(ji) * ld + int64_t(nq + hk) * d : nullptr, d, hf, k);
  load_row<DT>(ji < S ? base + int64_t(ji) * ld + int64_t(nq + nkv + hk) * d : nullptr, d, hf, v);
  f32x16 dk[DT], dv[DT];
  clear(dk);
  clear(dv);
  const int nb = (S - j0 + 31) / 32;  // query blocks of a head at or below the diagonal
  for (int it = wave; it < nb * heads; it += 4) {
    const int hq = hq0 + it / nb, i0 = j0 + (it % nb) * 32;
    const int64_t si = (int64_t(bi) * nq + hq) * S, row = int64_t(bi) * S + i0 + l32;
    const float *Q = base + int64_t(hq) * d, *dO = d_o + int64_t(bi) * S * ldd + int64_t(hq) * d;
    const bool live = i0 + l32 < S;
    float r[DT * 16], rc[16][DT], L[16], dl[16];
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int i = i0 + 8 * (e >> 2) + 4 * hf + (e & 3);
      L[e] = i < S ? lse[si + i] : 0.f;
      if (!TOGETHER) dl[e] = i < S ? delta[si + i] : 0.f;
    }
    load_row<DT>(live ? Q + int64_t(i0 + l32) * ld : nullptr, d, hf, r);
    f32x16 p = dot_rows(r, k);
    load_row<DT>(live ? dO + int64_t(i0 + l32) * ldd : nullptr, d, hf, r);
    if constexpr (TOGETHER) {
      float f[DT * 16], own = 0.f;  // of row i0 + l32
      load_row<DT>(live ? o + row * ldo + int64_t(hq) * d : nullptr, d, hf, f);
#pragma unroll
      for (int i = 0; i < DT * 16; i++) own += f[i] * r[i];
      own += __shfl_xor(own, 32, 64);
#pragma unroll
      for (int e = 0; e < 16; e++) dl[e] = __shfl(own, 8 * (e >> 2) + 4 * hf + (e & 3), 64);
    }
    load_cols<DT>(dO, ldd, i0, S, d, l32, hf, rc);
    f32x16 dp = dot_rows(r, v);
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int i = i0 + 8 * (e >> 2) + 4 * hf + (e & 3);
      p[e] = i >= ji && i < S ? __expf(p[e] * sc - L[e]) : 0.f;
      dp[e] = i >= ji && i < S ? p[e] * (dp[e] - dl[e]) : 0.f;  // dS
    }
    if (i0 > j0) accumulate<DT>(dv, rc, p);
    else accumulate_diagonal<DT>(dv, rc, p, dO, ldd, i0, S, d, l32, hf, lds.sp[wave], [&](int i) { return i >= ji; });
    load_cols<DT>(Q, ld, i0, S, d, l32, hf, rc);
    if (i0 > j0) accumulate<DT>(dk, rc, dp);
    else accumulate_diagonal<DT>(dk, rc, dp, Q, ld, i0, S, d, l32, hf, lds.sp[wave], [&](int i) { return i >= ji; });
  }
  sum_waves<DT>(dk, lds.part, wave, lane);
  sum_waves<DT>(dv, lds.part, wave, lane);
  if (wave != 0 || ji >= S) return;
  if (part) {
    float* out = part + ((int64_t(bi) * nq + hq0) * S + ji) * d;
    store_row<DT>(out, dk, sc, d, hf);
    store_row<DT>(out + int64_t(nb_all) * nq * S * d, dv, 1.f, d, hf);
    return;
  }
  float* out = dqkv + (int64_t(bi) * S + ji) * ldg;
  store_row<DT>(out + int64_t(nq + hk) * d, dk, sc, un, ji, d, hf);
  store_row<DT>(out + int64_t(nq + nkv + hk) * d, dv, 1.f, d, hf);
}

// One-dimensional grid: rank by rank of the blocks of 32, the longest first; in a rank the key blocks of every KV head (part: of every query
// head), then the query blocks; batch rows fastest.
template <int DT>
__global__ __launch_bounds__(256) void attn_bwd_f32_kernel(const float* __restrict__ qkv, int64_t ld, const float* __restrict__ o, int64_t ldo,
                                                           const float* __restrict__ lse, const float* __restrict__ d_o, int64_t ldd,
                                                           float* __restrict__ dqkv, int64_t ldg, int b, int S, int nq, int nkv, int d,
                                                           float* __restrict__ part, Unrotate un) {
  __shared__ BwdLds<DT> lds;
  const int kv = part ? nq : nkv, per = (kv + nq) * b, rank = blockIdx.x / per, x = blockIdx.x % per / b, bi = blockIdx.x % b;
  const int heads = part ? 1 : nq / nkv;
  if (x < kv) dkv_block<DT, true>(lds, rank * 32, x * heads, heads, bi, b, qkv, ld, o, ldo, lse, d_o, ldd, nullptr, dqkv, ldg, S, nq, nkv, d, part, un);
  else dq_block<DT, true>(lds, ((S + 31) / 32 - 1 - rank) * 32, x - kv, bi, qkv, ld, o, ldo, lse, d_o, ldd, nullptr, dqkv, ldg, S, nq, nkv, d, un);
}
// apart: grid as the forward's; and over (key blocks of 32, longest first; batch rows; KV heads)
template <int DT>
__global__ __launch_bounds__(256, DT <= 2 ? 2 : 1) void attn_dq_f32_kernel(const float* __restrict__ qkv, int64_t ld, const float* __restrict__ o, int64_t ldo,
                                                          const float* __restrict__ lse, const float* __restrict__ d_o, int64_t ldd,
                                                          float* __restrict__ delta, float* __restrict__ dqkv, int64_t ldg, int b, int S, int nq,
                                                          int nkv, int d, Unrotate un) {
  __shared__ BwdLds<DT> lds;
  dq_block<DT, false>(lds, ((S + 31) / 32 - 1 - blockIdx.x / nq / b) * 32, blockIdx.x % nq, blockIdx.x / nq % b, qkv, ld, o, ldo, lse, d_o, ldd, delta,
                      dqkv, ldg, S, nq, nkv, d, un);
}
template <int DT>
__global__ __launch_bounds__(256) void attn_dkv_f32_kernel(const float* __restrict__ qkv, int64_t ld, const float* __restrict__ lse,
                                                           const float* __restrict__ d_o, int64_t ldd, const float* __restrict__ delta,
                                                           float* __restrict__ dqkv, int64_t ldg, int b, int S, int nq, int nkv, int d, Unrotate un) {
  __shared__ BwdLds<DT> lds;
  const int grp = nq / nkv;
  dkv_block<DT, false>(lds, blockIdx.x / nkv / b * 32, blockIdx.x % nkv * grp, grp, blockIdx.x / nkv % b, b, qkv, ld, nullptr, 0, lse, d_o, ldd, delta,
                       dqkv, ldg, S, nq, nkv, d, nullptr, un);
}
// dK and dV from the parts of the query heads of a group, in ascending order; a thread owns four features and the four half a head on
__global__ __launch_bounds__(256) void gqa_reduce_f32_kernel(const float* __restrict__ part, int b, int S, int nq, int nkv, int d,
                                                             float* __restrict__ dqkv, int64_t ldg, Unrotate un) {
  const int64_t id = int64_t(blockIdx.x) * 256 + threadIdx.x, whole = int64_t(b) * nkv * S * (d / 8);
  if (id >= 2 * whole) return;
  const int what = id >= whole, grp = nq / nkv, half = d / 2;
  const int64_t r = what ? id - whole : id;
  const int c = int(r % (d / 8)) * 4, token = int(r / (d / 8) % S), hk = int(r / (d / 8) / S % nkv), bi = int(r / (d / 8) / S / nkv);
  const float* p = part + (((int64_t(what) * b + bi) * nq + hk * grp) * S + token) * d + c;
  auto at4 = [](const float* q) { return *reinterpret_cast<const float4*>(q); };
  float4 x = at4(p), y = at4(p + half);
  for (int i = 1; i < grp; i++) {
    const float4 u = at4(p + int64_t(i) * S * d), v = at4(p + int64_t(i) * S * d + half);
    x.x += u.x; x.y += u.y; x.z += u.z; x.w += u.w;
    y.x += v.x; y.y += v.y; y.z += v.z; y.w += v.w;
  }
  if (!what && un.cos_tab) {
    const float4 cs = at4(un.cos_tab + int64_t(token) * half + c), sn = at4(un.sin_tab + int64_t(token) * half + c), u = x, v = y;
    x = make_float4(u.x * cs.x + v.x * sn.x, u.y * cs.y + v.y * sn.y, u.z * cs.z + v.z * sn.z, u.w * cs.w + v.w * sn.w);
    y = make_float4(v.x * cs.x - u.x * sn.x, v.y * cs.y - u.y * sn.y, v.z * cs.z - u.z * sn.z, v.w * cs.w - u.w * sn.w);
  }
  float* out = dqkv + (int64_t(bi) * S + token) * ldg + int64_t(nq + (what ? nkv : 0) + hk) * d + c;
  *reinterpret_cast<float4*>(out) = x;
  *reinterpret_cast<float4*>(out + half) = y;
}

template <class F>
hipError_t for_tiles(int d, F&& f) {
  if (d <= 32) f(std::integral_constant<int, 1>{});
  else if (d <= 64) f(std::integral_constant<int, 2>{});
  else if (d <= 96) f(std::integral_constant<int, 3>{});
  else f(std::integral_constant<int, 4>{});
  return hipGetLastError();
}

}  // namespace

namespace mls {

// head_dim a multiple of 16 up to 128; row strides multiples of 8, 16-byte aligned buffers
hipError_t attn_fwd_f32(const void* qkv, int64_t ld_qkv, void* o, int64_t ld_o, float* lse, int b, int S, int nq, int nkv,
                        int d, hipStream_t st) {
  if (b == 0 || S == 0 || nq == 0) return hipSuccess;
  return for_tiles(d, [&](auto DT) {
    hipLaunchKernelGGL(attn_fwd_f32_kernel<decltype(DT)::value>, dim3(unsigned((S + 31) / 32) * nq * b), dim3(256), 0, st,
                       (const float*)qkv, ld_qkv, (float*)o, ld_o, lse, b, S, nq, nkv, d);
  });
}

// dQ, dK and dV in one launch, by blocks of 32 query rows, a workgroup each and as many for the key rows; a CU has a place for one.  Many more of
// them than places balance by themselves, and then the rows of O that the dK / dV part reads for delta, and the registers that part costs the
// other, outweigh what the balance gains; so do two rounds of short chains instead of one for either part.  Backward, us, apart / together:
//   d <= 64: 250 blocks (1598 positions) 165 / 107, 246 (176) 38.7 / 37.7 but 252 (100) 26.4 / 28.9, 384 (252) 59 / 53, 400 (1592) 112 / 121, 456 (58) 43.5 / 48.3,
//            483 (203) 34.6 / 40.2; wider: 265 (150) 110 / 75, 270 (1410) 360 / 287, 300 (633) 185 / 200, 364 (210) 143 / 119, 425 (796) 268 / 319,
//            476 of 80 (888) 170 / 199, 516 of 112 (115) 162 / 122
//   grouped: 24 heads over 12 at 700 positions (528 blocks) 145 / 123, 22 over 11 of 112 at 856 (594) 400 / 584, 2 x 64 over 32 at 118 (512) 23.5 / 26.2
bool bwd_f32_together(int b, int S, int nq, int nkv, int d) {
  const int64_t n = (S + 31) / 32, q = int64_t(b) * nq * n, k = int64_t(b) * nkv * n;
  if (nq > nkv) return q <= 544 && (k < 256 || n > 4);
  if (q > 180 && q <= 256 && n <= 4) return false;
  if (d <= 64) return q <= 384;
  return q <= 288 || (d <= 96 ? q <= 400 && n <= 8 : q <= 544 && n <= 12);
}
// The query heads of a group apart where that shortens a chain of key blocks by more than the additional workgroups and the sum cost: us, in one
// workgroup / apart: 8 heads over 1 at 563 positions (144 blocks, chains of 18 blocks x 8 heads) 297 / 55, 4 over 1 at 437 (448, 56) 122 / 83, 2
// over 1 at 246 (16, 16) 40.6 / 26.9 but at 38 (168, 4) 9.1 / 16.1, 42 (384, 4) 28.4 / 39.9, 4 over 1 at 83 (480, 12) 34 / 54.  A float of workspace per
// element of dK and dV and query head.
size_t attn_bwd_f32_scratch_floats(int b, int S, int nq, int nkv, int d) {
  const int64_t n = (S + 31) / 32, q = int64_t(b) * nq * n, chain = n * (nq / nkv);
  const bool apart = nq > nkv && chain > 4 && (q <= 180 || 16 * chain >= q) && int64_t(b) * nkv * n < 256;
  return apart && bwd_f32_together(b, S, nq, nkv, d) ? size_t(2) * b * nq * S * d : 0;
}

hipError_t attn_bwd_f32(const void* qkv, int64_t ld_qkv, const void* o, int64_t ld_o, const float* lse, const void* d_o,
                        int64_t ld_do, void* dqkv, int64_t ld_dqkv, float* delta, int b, int S, int nq, int nkv, int d, hipStream_t st, float* part,
                        const float* cos_tab, const float* sin_tab) {
  if (b == 0 || S == 0 || nq == 0) return hipSuccess;
  if (!attn_bwd_f32_scratch_floats(b, S, nq, nkv, d)) part = nullptr;
  const unsigned n = unsigned((S + 31) / 32);
  const Unrotate un = {cos_tab, sin_tab};
  return for_tiles(d, [&](auto DTC) {
    constexpr int DT = decltype(DTC)::value;
    if (!bwd_f32_together(b, S, nq, nkv, d)) {
      hipLaunchKernelGGL(attn_dq_f32_kernel<DT>, dim3(n * nq * b), dim3(256), 0, st, (const float*)qkv, ld_qkv, (const float*)o, ld_o, lse,
                         (const float*)d_o, ld_do, delta, (float*)dqkv, ld_dqkv, b, S, nq, nkv, d, un);
      hipLaunchKernelGGL(attn_dkv_f32_kernel<DT>, dim3(n * nkv * b), dim3(256), 0, st, (const float*)qkv, ld_qkv, lse, (const float*)d_o, ld_do, delta,
                         (float*)dqkv, ld_dqkv, b, S, nq, nkv, d, un);
      return;
    }
    hipLaunchKernelGGL(attn_bwd_f32_kernel<DT>, dim3(n * ((part ? nq : nkv) + nq) * b), dim3(256), 0, st, (const float*)qkv, ld_qkv, (const float*)o,
                       ld_o, lse, (const float*)d_o, ld_do, (float*)dqkv, ld_dqkv, b, S, nq, nkv, d, part, un);
    if (part)
      hipLaunchKernelGGL(gqa_reduce_f32_kernel, dim3(unsigned((int64_t(2) * b * nkv * S * (d / 8) + 255) / 256)), dim3(256), 0, st, part, b, S, nq,
                         nkv, d, (float*)dqkv, ld_dqkv, un);
  });
}

}  // namespace mls
