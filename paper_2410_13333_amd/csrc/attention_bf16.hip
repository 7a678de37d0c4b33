// Causal grouped-query attention for bf16 storage on the gfx950 matrix cores: forward with online softmax,
// backward as two kernels (dQ, which also forms the row sums delta = dO . O; dK and dV) that recompute the
// probabilities from the saved log-sum-exp.  Where few workgroups share the chip, both run in one launch (bwd_together), or dQ is formed
// from the dS that the dK / dV kernel leaves behind instead (dq_from_ds); nothing else of size S x S is ever written.  No float atomics, so results are
// bitwise reproducible.
//
// Register-resident probabilities.  v_mfma_f32_32x32x16_bf16 leaves element (g*4+r) of lane l at
// [row (l/32)*4 + 8g + r][col l%32] of the 32x32 result and expects the B operand as "lane l holds column
// l%32, eight k-values".  All score-like products are therefore computed TRANSPOSED so that the softmax row
// index is the lane's column: a lane then owns all the probabilities of its row that it computed, can turn
// them into a B operand of the next product without leaving its registers, and keeps the running row
// maximum / sum as plain scalars.  The contraction index of that next product is permuted (k-values
// 4g..4g+3 and 8+4g..8+4g+3 per 16-step), which is free because the A operand is fetched with the same
// permutation by ds_read_b64_tr_b16 out of a tile stored [kv][d] just as it lies in memory.
//
// LDS tiles are 64 rows x D columns, unpadded, with an XOR swizzle of the 16-byte chunks that makes both
// access patterns bank-conflict free: ds_read_b128 of 16 consecutive rows at one column chunk, and the
// transposing 8-byte reads of 4 consecutive rows x 64 bytes.
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"

namespace {

// 16 bytes per lane from a raw buffer straight into LDS (64 lanes fill 1 KiB at lds_byte); out-of-range lanes
// are zero-filled.  Inline asm so that the waits are placed by hand (see gemm_bf16_t16.hip).
__device__ __forceinline__ void dma16(i32x4 rsrc, uint32_t voff, uint32_t lds_byte) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_byte), "v"(voff), "s"(rsrc)
               : "memory");
}
// the same with 4 bytes per lane (256 bytes at lds_byte)
__device__ __forceinline__ void dma4(i32x4 rsrc, uint32_t voff, uint32_t lds_byte) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds_byte), "v"(voff), "s"(rsrc)
               : "memory");
}
__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

constexpr int AT_THREADS = 256;
constexpr int TR = 64;  // rows of an LDS tile
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// element offset of (row, col) inside a swizzled 64 x D tile
template <int D>
__device__ __forceinline__ int toff(int row, int col) {
  if (D == 128) {
    const int sw = ((row & 3) << 2) | ((row >> 2) & 3);
    return row * 128 + ((((col >> 3) ^ sw)) << 3) + (col & 7);
  } else {
    const int line = row >> 1;
    const int sw = ((line & 1) << 2) | ((line >> 1) & 3);
    return line * 128 + (((((row & 1) << 3) | (col >> 3)) ^ sw) << 3) + (col & 7);
  }
}

template <int D, int ROWS = TR>
struct Tile {
  static constexpr int BYTES = ROWS * D * 2;
  static constexpr int NI = BYTES / 1024 / 4;  // DMA instructions per wave per tile
  // Per-lane source offsets (bytes, relative to element (row0, col0) of the source matrix) of this wave's DMA
  // instructions: instruction q = wave*NI + i fills LDS bytes [1024 q, 1024 q + 1024) of the tile, and the lane
  // that writes a given 16-byte slot fetches the chunk the swizzle assigns to it.
  uint32_t off[NI];
  __device__ __forceinline__ void init(int64_t ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NI; i++) {
      const int q = wave * NI + i;
      int row, chunk;
      if (D == 128) {
        row = q * 4 + (lane >> 4);
        chunk = (lane & 15) ^ (((row & 3) << 2) | ((row >> 2) & 3));
      } else {
        const int line = q * 4 + (lane >> 4);
        const int idx = (lane & 15) ^ (((line & 1) << 2) | ((line >> 1) & 3));
        row = line * 2 + (idx >> 3);
        chunk = idx & 7;
      }
      off[i] = uint32_t((int64_t(row) * ld + chunk * 8) * 2);
    }
  }
  // the same from a matrix of `rows` rows at `m` (row stride ld): everything that changes is in the scalar descriptor
  __device__ __forceinline__ void dma(const bf16_t* m, int64_t ld, int row0, int rows, uint32_t tile, int wave) const {
    const i32x4 src = make_rsrc(m + int64_t(row0) * ld, row0 < rows ? uint32_t((int64_t(rows - row0) * ld) * 2) : 0u);
#pragma unroll
    for (int i = 0; i < NI; i++) dma16(src, off[i], tile + (wave * NI + i) * 1024);
  }
  // rows [row0, row0+64) x cols [col0, col0+D) of the matrix behind rsrc (row stride ld) -> tile at LDS byte
  // address `tile`; rows at or beyond the end of the buffer are zero-filled; live = false sends nothing useful
  __device__ __forceinline__ void dma(i32x4 rsrc, int64_t ld, int row0, int col0, uint32_t tile, int wave,
                                      bool live) const {
    const uint32_t base = uint32_t((int64_t(row0) * ld + col0) * 2);
#pragma unroll
    for (int i = 0; i < NI; i++) dma16(rsrc, live ? base + off[i] : OOB, tile + (wave * NI + i) * 1024);
  }
  // A operand, rows = tile rows rt*32 .. +31, k = tile columns kk*16 .. +15
  static __device__ __forceinline__ bf16x8 frag_rows(const bf16_t* t, int rt, int kk, int lane) {
    const uint4 v = *reinterpret_cast<const uint4*>(t + toff<D>(rt * 32 + (lane & 31), kk * 16 + (lane >> 5) * 8));
    return __builtin_bit_cast(bf16x8, v);
  }
  // A operand, rows = tile COLUMNS ct*32 .. +31, k = tile rows of the 16-step `ks` in the permuted order
  // that matches a B operand built from accumulator registers: k-values 4g..4g+3 then 8+4g..8+4g+3, g = lane/32.
  static __device__ __forceinline__ bf16x8 frag_cols(const bf16_t* t, int ct, int ks, int lane) {
    const int row = ks * 16 + (lane >> 5) * 4 + ((lane & 15) >> 2);
    const int col = ct * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)(t + toff<D>(row, col)));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)(t + toff<D>(row + 8, col)));
    s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
};

// Fragment reads of swizzled tiles whose place in LDS is a compile-time constant: one address per fragment column (the
// swizzle turns a step along the columns into an XOR of the address), everything else in the read's immediate offset.
template <int D>
struct Frags {
  uint32_t r[D / 16], lo[D / 32], hi[D / 32];
  __device__ __forceinline__ void init(uint32_t lds0, int lane) {
    const uint32_t br = lds0 + toff<D>(lane & 31, (lane >> 5) * 8) * 2;
    const uint32_t bc = lds0 + toff<D>((lane >> 5) * 4 + ((lane & 15) >> 2), ((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
#pragma unroll
    for (int i = 0; i < D / 16; i++) r[i] = br ^ (i << 5);
#pragma unroll
    for (int i = 0; i < D / 32; i++) {
      lo[i] = bc ^ (i << 6);
      hi[i] = bc ^ (i << 6) ^ 32;
    }
  }
  // the other buffer of a pair (the first one at a multiple of twice the tile size)
  __device__ __forceinline__ void flip_rows() {
#pragma unroll
    for (int i = 0; i < D / 16; i++) r[i] ^= TR * D * 2;
  }
  __device__ __forceinline__ void move_cols(uint32_t by) {
#pragma unroll
    for (int i = 0; i < D / 32; i++) {
      lo[i] += by;
      hi[i] += by;
    }
  }
  // A operand, rows = tile rows rt*32 .. +31, k = tile columns kk*16 .. +15; tile: its byte offset from lds0
  template <int TILE, int RT>
  __device__ __forceinline__ bf16x8 rows(int kk) const {
    return *(const MLS_LDS bf16x8*)(r[kk] + (TILE + RT * 32 * D * 2));
  }
  // A operand, rows = tile COLUMNS ct*32 .. +31, k = tile rows of the 16-step KS in the permuted order that matches a B
  // operand built from accumulator registers: k-values 4g..4g+3 then 8+4g..8+4g+3, g = lane/32
  template <int TILE, int KS>
  __device__ __forceinline__ bf16x8 cols(int ct) const {
    s16x4 l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)(lo[ct] + (TILE + KS * 16 * D * 2)));
    s16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)(hi[ct] + (TILE + KS * 16 * D * 2 + 8 * D * 2)));
    s16x8 v = {l[0], l[1], l[2], l[3], h[0], h[1], h[2], h[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
};

// B operand straight from global memory: column l%32 = matrix row row0 + l%32, k = matrix columns kk*16 + (l/32)*8 ..
__device__ __forceinline__ bf16x8 gfrag(const bf16_t* __restrict__ g, int64_t ld, int row, int col, bool valid) {
  uint4 v = make_uint4(0, 0, 0, 0);
  if (valid) v = *reinterpret_cast<const uint4*>(g + int64_t(row) * ld + col);
  return __builtin_bit_cast(bf16x8, v);
}

// two accumulator groups (2s, 2s+1) of a 32x32 result -> B operand of the next product
__device__ __forceinline__ bf16x8 acc_to_b(const f32x16& a, int s) {
  uint4 v;
  v.x = pack_bf16x2(a[8 * s + 0], a[8 * s + 1]);
  v.y = pack_bf16x2(a[8 * s + 2], a[8 * s + 3]);
  v.z = pack_bf16x2(a[8 * s + 4], a[8 * s + 5]);
  v.w = pack_bf16x2(a[8 * s + 6], a[8 * s + 7]);
  return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int e = 0; e < 16; e++) z[e] = 0.f;
  return z;
}

// maximum of a lane and its partner in the other half of the wavefront, without a trip through LDS
__device__ __forceinline__ float max_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// N LDS fragment reads feeding N MFMAs, each read issued DEPTH fragments ahead of its use so that the LDS latency
// hides behind the MFMAs in between (left to itself the compiler reads every fragment right before its MFMA and
// waits for it).  read(i) returns fragment i (RPF LDS instructions each), use(i, f) issues the MFMA that takes it.
template <int N, int DEPTH, int RPF, class Read, class Use>
__device__ __forceinline__ void read_ahead(Read&& read, Use&& use) {
  bf16x8 f[N];  // fully unrolled: a fragment's registers are free again once its MFMA has issued
#pragma unroll
  for (int i = 0; i < DEPTH && i < N; i++) f[i] = read(i);
#pragma unroll
  for (int i = 0; i < N; i++) {
    if (i + DEPTH < N) f[i + DEPTH] = read(i + DEPTH);
    use(i, f[i]);
  }
  // the issue order the scheduler is asked for: DEPTH fragments, then MFMA / next fragment alternating
#pragma unroll
  for (int i = 0; i < DEPTH && i < N; i++) __builtin_amdgcn_sched_group_barrier(0x100, RPF, 0);
#pragma unroll
  for (int i = 0; i < N; i++) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (i + DEPTH < N) __builtin_amdgcn_sched_group_barrier(0x100, RPF, 0);
  }
}

// store a transposed 32x32 result (col l%32 = token, rows = feature index) as bf16: 4 consecutive features = 8 bytes
__device__ __forceinline__ void store_t(bf16_t* __restrict__ out, int64_t ld, int token, int col0, const f32x16& a,
                                        float mul, int lane, bool valid) {
  if (!valid) return;
#pragma unroll
  for (int g = 0; g < 4; g++) {
    uint2 v;
    v.x = pack_bf16x2(a[g * 4 + 0] * mul, a[g * 4 + 1] * mul);
    v.y = pack_bf16x2(a[g * 4 + 2] * mul, a[g * 4 + 3] * mul);
    *reinterpret_cast<uint2*>(out + int64_t(token) * ld + col0 + (lane >> 5) * 4 + 8 * g) = v;
  }
}

// The same store for a whole head vector of a gradient w.r.t. rotated q or k, turned back by the rotary angle of
// its position on the way out (the transpose of the forward rotation): with (g1, g2) the halves of the gradient,
// the result is (g1 c + g2 s, g2 c - g1 s).  Feature i of the first half sits in tile i / 32, its partner
// i + D/2 in tile i / 32 + D/64, same register.  cos_tab, sin_tab: [S][D/2] fp32; pos: position in the sequence.
template <int D>
__device__ __forceinline__ void store_t_unrotate(bf16_t* __restrict__ out, int64_t ld, int token, int pos, int col0,
                                                 const f32x16 (&a)[D / 32], float mul, const float* __restrict__ cos_tab,
                                                 const float* __restrict__ sin_tab, int lane, bool valid) {
  if (!valid) return;
  constexpr int H = D / 64, D2 = D / 2;
#pragma unroll
  for (int t = 0; t < H; t++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int f = t * 32 + (lane >> 5) * 4 + 8 * g;
      const float4 c = *reinterpret_cast<const float4*>(cos_tab + int64_t(pos) * D2 + f);
      const float4 sn = *reinterpret_cast<const float4*>(sin_tab + int64_t(pos) * D2 + f);
      const float cs[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
      float o1[4], o2[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const float g1 = a[t][g * 4 + r] * mul, g2 = a[t + H][g * 4 + r] * mul;
        o1[r] = g1 * cs[r] + g2 * ss[r];
        o2[r] = g2 * cs[r] - g1 * ss[r];
      }
      uint2 v1, v2;
      v1.x = pack_bf16x2(o1[0], o1[1]); v1.y = pack_bf16x2(o1[2], o1[3]);
      v2.x = pack_bf16x2(o2[0], o2[1]); v2.y = pack_bf16x2(o2[2], o2[3]);
      *reinterpret_cast<uint2*>(out + int64_t(token) * ld + col0 + f) = v1;
      *reinterpret_cast<uint2*>(out + int64_t(token) * ld + col0 + D2 + f) = v2;
    }
}

// ================================================================ forward
// grid (n_q, q blocks of 128, b) with the longest query blocks dispatched first over all heads; wave w owns
// query rows q0 + 32w .. +31; loops over KV blocks of 64 = two sub-blocks of 32 keys.  Two workgroups fit a CU.
//
// What bounded it was one wavefront's chain scores -> softmax -> product with V: the matrix pipe was busy 44 % of the
// time with two wavefronts per SIMD.  The chain is therefore software-pipelined over the sub-blocks: a step issues the
// 16 MFMAs of one sub-block's S = K Q^T and of another's O += V^T P, neither of which needs the softmax whose vector
// instructions go out in between (about five fit behind one MFMA).  S runs two sub-blocks ahead of the softmax, so that the
// maximum is taken over a block of 64 keys at once and the accumulators are rescaled once per block at most, and P V runs one
// behind it.  K has two buffers, V three; the one barrier per block frees those of K(u-1) and V(u-3).
// Measured (us, unpipelined -> this): 4096 positions, 32 heads of 128: 163 -> 160; 2048, 16 of 128 (one workgroup per CU,
// where the chain is everything): 60 -> 47.5; 4096, 16 of 128: 117 -> 100; 4096, 16 of 64: 85 -> 62.  Every bit of the result
// is the unpipelined kernel's.  With every CU full the vector instructions and the MFMAs of a SIMD take about nine tenths of the
// cycles one after the other.
template <int D>
__global__ __launch_bounds__(AT_THREADS, 2) void attn_fwd_kernel(const bf16_t* __restrict__ qkv, int64_t ld, bf16_t* __restrict__ o, int64_t ldo,
                                                                 float* __restrict__ lse, int S, int nq, int nkv) {
  using TL = Tile<D>;
  constexpr int KD = D / 16, DT = D / 32, FA = 6, NV = 5;  // reads ahead; vector instructions per MFMA
  __shared__ __attribute__((aligned(4 * TR * D))) bf16_t lds[5][TR * D];  // two buffers of K, three of V
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qb = gridDim.y - 1 - blockIdx.y;  // longest rows first
  const int hq = blockIdx.x, bi = blockIdx.z, hk = hq / (nq / nkv);
  const bf16_t* base = qkv + int64_t(bi) * S * ld;
  const int q0 = qb * 128, qw = q0 + wave * 32, qi = qw + (lane & 31);
  const float sc = rsqrtf((float)D) * LOG2E;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MLS_LDS bf16_t*)&lds[0][0];
  TL tl;
  tl.init(ld, wave, lane);
  Frags<D> fr;
  fr.init(lds0, lane);
  const bf16_t *kp = base + (nq + hk) * D, *vp = kp + nkv * D;
  const int nblk = (min(S, q0 + 128) + TR - 1) / TR;  // KV blocks of the workgroup
  // blocks beyond the last one are requested as empty
  auto issue_k = [&](int u) { tl.dma(kp, ld, u * TR, u < nblk ? S : 0, lds0 + (u & 1) * TL::BYTES, wave); };
  auto issue_v = [&](int u) { tl.dma(vp, ld, u * TR, u < nblk ? S : 0, lds0 + (2 + u % 3) * TL::BYTES, wave); };

  bf16x8 qf[KD];
#pragma unroll
  for (int kk = 0; kk < KD; kk++) qf[kk] = gfrag(base, ld, qi, hq * D + kk * 16 + (lane >> 5) * 8, qi < S);

  f32x16 acc[DT];
#pragma unroll
  for (int t = 0; t < DT; t++) acc[t] = zero16();
  float m = -INFINITY, l = 0.f;
  f32x16 st[2] = {zero16(), zero16()}, nx[2];  // S of the block whose softmax comes next, and of the one after it
  bf16x8 pf[2][2] = {};                        // P of the two sub-blocks

  const int diag = qw >> 5;                           // the sub-block on this wavefront's diagonal; later ones are masked
  const int nw = min(diag / 2 + 1, nblk);             // KV blocks this wavefront needs; only the last one has masked pairs
  float ps = 0.f;

  // One step.  DO_S: S of sub-block H of the current K tile, into nx[H].  DO_SM: the exponentials of sub-block H of the block in
  // `st`; with H = 0 that block's maximum before, and the reference moves (BLK: its index, for the mask).  DO_PV: O += V^T P of
  // the other sub-block, the one before in order.
  auto step = [&](auto HC, auto DO_S, auto DO_SM, auto MASK, int blk, auto DO_PV) {
    constexpr int KT = 0, VT = 2 * TL::BYTES, H = decltype(HC)::value;
    constexpr bool do_s = decltype(DO_S)::value, do_sm = decltype(DO_SM)::value, do_pv = decltype(DO_PV)::value;
    // MFMAs in their order: S and PV alternate (KD of each; S is one chain), each fragment read FA MFMAs ahead
    f32x16 sn = zero16();
    constexpr int NM = KD * (do_s + do_pv);
    auto is_s = [](int i) constexpr { return do_s && (!do_pv || !(i & 1)); };
    bf16x8 f[NM > 0 ? NM : 1];
    auto read = [&](auto IC) {
      constexpr int i = decltype(IC)::value, q = do_s && do_pv ? i / 2 : i;
      if constexpr (is_s(i)) f[i] = fr.template rows<KT, H>(q);
      else f[i] = fr.template cols<VT, (1 - H) * 2 + q / DT>(q % DT);
    };
    static_for<(FA < NM ? FA : NM)>(read);
    static_for<NM>([&](auto IC) {
      constexpr int i = decltype(IC)::value, q = do_s && do_pv ? i / 2 : i;
      if constexpr (is_s(i)) sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], qf[q], sn, 0, 0, 0);
      else acc[q % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], pf[1 - H][q / DT], acc[q % DT], 0, 0, 0);
      if constexpr (i + FA < NM) read(std::integral_constant<int, i + FA>{});
    });
    float mn = m;
    if constexpr (do_sm) {
      if constexpr (H == 0) {
        // row maximum of the raw scores (the scale is positive: it commutes with the maximum and is folded into the
        // exponent below); the mask arithmetic is compiled only into the diagonal path
        float mx = -INFINITY;
#pragma unroll
        for (int jt = 0; jt < 2; jt++) {
          const int lim = qi - blk * 64 - jt * 32 - (lane >> 5) * 4;  // key 8 (e / 4) + e % 4 of this lane's half is masked beyond it
#pragma unroll
          for (int e = 0; e < 16; e++) {
            if (decltype(MASK)::value && 8 * (e >> 2) + (e & 3) > lim) st[jt][e] = -INFINITY;
            mx = fmaxf(mx, st[jt][e]);
          }
        }
        mx = max_halves(mx);
        // The reference of the exponents is the row's maximum itself, as far as it is known, so that the largest probability of
        // a row is 1 and stays exact when P is rounded to bf16.  A reference that only follows when the maximum has passed it
        // by a margin saves most of the rescaling below, but then the row's largest term carries a rounding error of 2^-9 like
        // the others: on rows that look at few keys that is most of the error.
        mn = fmaxf(m, mx * sc);  // finite: block 0 always holds j = 0 <= i
        ps = 0.f;
      }
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const float p = __builtin_amdgcn_exp2f(st[H][e] * sc - mn);
        st[H][e] = p;
        ps += p;
      }
      pf[H][0] = acc_to_b(st[H], 0);
      pf[H][1] = acc_to_b(st[H], 1);
      asm volatile("" : "+v"(pf[H][0]), "+v"(pf[H][1]), "+v"(ps));  // here, between the MFMAs, and not behind the branch below
      if constexpr (do_s && do_pv) {
        static_for<FA>([&](auto IC) { __builtin_amdgcn_sched_group_barrier(0x100, is_s(decltype(IC)::value) ? 1 : 2, 0); });
        static_for<NM>([&](auto IC) {
          constexpr int i = decltype(IC)::value;
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if constexpr (i + FA < NM) __builtin_amdgcn_sched_group_barrier(0x100, is_s(i + FA) ? 1 : 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x402, NV, 0);
        });
      }
      if constexpr (H == 0) {
        if (__any(mn > m)) {  // rescale only when some row's maximum moved
          const float corr = __builtin_amdgcn_exp2f(m - mn);
          l *= corr;
#pragma unroll
          for (int t = 0; t < DT; t++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[t][e] *= corr;
          m = mn;
        }
      } else {
        l += ps;
      }
    }
    if constexpr (do_s) nx[H] = sn;
    if constexpr (H == 1) {
      st[0] = nx[0];
      st[1] = nx[1];
    }
  };
  using Y = std::true_type;
  using N = std::false_type;
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  // every wavefront passes nblk + 1 barriers: block 0, its blocks, its last softmax, and the blocks that only later rows need
  auto next = [&](int u) {
    wait_dma();       // this wave's part of K(u), V(u-1) has landed ...
    __syncthreads();  // ... and so has everyone's; all reads of K(u-1), V(u-3) are retired
    issue_k(u + 1);
    issue_v(u);
  };
  int vs = 0;  // V's buffer
  auto next_v = [&]() {
    vs = vs == 2 ? 0 : vs + 1;
    fr.move_cols(vs == 0 ? 0u - 2 * TL::BYTES : TL::BYTES);
  };
  nx[0] = nx[1] = zero16();
  issue_k(0);
  next(0);
  step(C0{}, Y{}, N{}, N{}, 0, N{});
  step(C1{}, Y{}, N{}, N{}, 0, N{});
  if (nw > 1) {
    next(1);
    fr.flip_rows();
    step(C0{}, Y{}, Y{}, N{}, 0, N{});
    step(C1{}, Y{}, Y{}, N{}, 0, Y{});
    for (int u = 2; u < nw; u++) {
      next(u);
      fr.flip_rows();
      step(C0{}, Y{}, Y{}, N{}, u - 1, Y{});
      next_v();
      step(C1{}, Y{}, Y{}, N{}, u - 1, Y{});
    }
    next(nw);
    step(C0{}, N{}, Y{}, Y{}, nw - 1, Y{});
    next_v();
  } else {
    next(1);
    step(C0{}, N{}, Y{}, Y{}, 0, N{});
  }
  step(C1{}, N{}, Y{}, N{}, nw - 1, Y{});
  step(C0{}, N{}, N{}, N{}, 0, Y{});
  for (int u = nw + 1; u <= nblk; u++) next(u);
  wait_dma();
  l += __shfl_xor(l, 32, 64);
  const float inv = 1.f / l;
  bf16_t* ob = o + int64_t(bi) * S * ldo;
#pragma unroll
  for (int t = 0; t < DT; t++) store_t(ob, ldo, qi, hq * D + t * 32, acc[t], inv, lane, qi < S);
  if (lane < 32 && qi < S) lse[(int64_t(bi) * nq + hq) * S + qi] = (m + __builtin_amdgcn_logf(l)) * LN2;
}

// ---------------------------------------------------------------- forward, few workgroups
// grid (n_q b, q blocks of 64), longest first.  Wave w owns query rows q0 + 32 (w / 2) .. +31 and, of every block of 64 keys, the
// sub-block w % 2: half the chain of the kernel above for twice the workgroups.  The two partial softmaxes of a row meet in LDS at the end.
//
// What bounds it is a wavefront's issue: about 100 vector instructions, 16 of them exponentials, and 16 products per sub-block, 0.65 us,
// whether it is alone on its SIMD or not.  The pipeline is therefore one of sub-blocks, two iterations per turn of the loop so that every
// buffer and every fragment address is a constant, in exactly the order written: products with V of the block before the last on both
// sides of the barrier, whose fragments were read an iteration before, so that neither the barrier nor the first reads behind it are waited for.
// Measured (us, the kernel above -> this): 2048 positions, 16 heads of 128: 45.4 -> 32.0; 1024, 16: 23.7 -> 15.8; 512, 16: 13.5 -> 10.0;
// 4096, 8: 80 -> 54; 3000, 4: 57 -> 33; 2 x 1000, 16 of 64: 17.4 -> 12.4; 512, 16 of 64: 9.9 -> 7.3.  (With a wait for the rows of Q left to
// the compiler, which put it into the loop: 34.8, 16.8, 10.5, 58.9, 35.9, 13.1, 7.7.)
template <int D>
__global__ __launch_bounds__(AT_THREADS, 2) void attn_fwd_pair_kernel(const bf16_t* __restrict__ qkv, int64_t ld, bf16_t* __restrict__ o, int64_t ldo,
                                                                      float* __restrict__ lse, int S, int nq, int nkv) {
  using TL = Tile<D>;
  constexpr int KD = D / 16, DT = D / 32, B = TL::BYTES, KA = 4;  // KA: fragments of K read ahead
  __shared__ __attribute__((aligned(4 * TR * D))) bf16_t lds[4][TR * D];  // two buffers of K, two of V
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kh = wave & 1;
  const int qb = gridDim.y - 1 - blockIdx.y;  // longest rows first
  const int hq = blockIdx.x % nq, bi = blockIdx.x / nq, hk = hq / (nq / nkv);
  const bf16_t* base = qkv + int64_t(bi) * S * ld;
  const int q0 = qb * 64, qw = q0 + (wave >> 1) * 32, qi = qw + (lane & 31);
  const float sc = rsqrtf((float)D) * LOG2E;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MLS_LDS bf16_t*)&lds[0][0];
  TL tl;
  tl.init(ld, wave, lane);
  Frags<D> fr;
  fr.init(lds0 + kh * (32 * D * 2), lane);  // (the swizzle repeats after 16 rows)
  const int nblk = (min(S, q0 + 64) + TR - 1) / TR;
  const uint32_t blk_bytes = uint32_t(TR * ld * 2), rec = uint32_t(int64_t(min(S, nblk * TR)) * ld * 2);
  i32x4 rk = make_rsrc(base + (nq + hk) * D, rec), rv = make_rsrc(base + (nq + nkv + hk) * D, rec);
  const uint32_t dst = lds0 + wave * TL::NI * 1024;
  // the next block of K (V) into buffer `buf`
  auto issue = [&](i32x4& r, int buf) {
#pragma unroll
    for (int i = 0; i < TL::NI; i++) dma16(r, tl.off[i], dst + buf * B + i * 1024);
    const uint64_t a = ((uint64_t)(uint32_t)r[1] << 32 | (uint32_t)r[0]) + blk_bytes;
    r[0] = (int)(uint32_t)a;
    r[1] = (int)(uint32_t)(a >> 32);
    r[2] = max(r[2] - (int)blk_bytes, 0);
  };

  bf16x8 qf[KD];
#pragma unroll
  for (int kk = 0; kk < KD; kk++) qf[kk] = gfrag(base, ld, qi, hq * D + kk * 16 + (lane >> 5) * 8, qi < S);
  f32x16 acc[DT];
#pragma unroll
  for (int t = 0; t < DT; t++) acc[t] = zero16();
  float m = -3e38f, l = 0.f;  // (finite: a wavefront may have no key at all)
  f32x16 st[2];               // scores of a block, by its parity
  bf16x8 pf[2][2];            // and its probabilities
  bf16x8 vf[KD], kf[KD];      // fragments of V of block u - 2 and of K of block u
#pragma unroll
  for (int n = 0; n < KD; n++) vf[n] = bf16x8{};
  pf[0][0] = pf[0][1] = pf[1][0] = pf[1][1] = bf16x8{};
  // the compiler's own wait for the rows of Q, here and not in the loop, where it would be one for the requests of the next block
#pragma unroll
  for (int kk = 0; kk < KD; kk++) asm volatile("" : "+v"(qf[kk]));

  // An iteration: O += V^T P of the block before the last, the exponentials of the last one, S of the next one, whose parity is P; in
  // exactly the order written.  MASK: the last block is the one on the diagonal.
  auto iter = [&](auto PC, auto DO_S, auto DO_SM, auto MASK, auto DO_PV) {
    constexpr int P = decltype(PC)::value, Q = 1 - P;
    constexpr bool do_s = decltype(DO_S)::value, do_sm = decltype(DO_SM)::value, do_pv = decltype(DO_PV)::value;
    float mx = -INFINITY, mn = m, ps = 0.f;
    constexpr int H = KD / 2;  // products before the barrier, and slots of the maximum
    // softmax work of slot n (of 2 KD)
    auto between = [&](auto NC) {
      constexpr int n = decltype(NC)::value;
      if constexpr (do_sm) {
        if constexpr (n < H) {
          if constexpr (n == 0 && decltype(MASK)::value) {
            const int lim = qi - q0 - kh * 32 - (lane >> 5) * 4;
#pragma unroll
            for (int e = 0; e < 16; e++)
              if (8 * (e >> 2) + (e & 3) > lim) st[Q][e] = -INFINITY;
          }
#pragma unroll
          for (int e = 16 * n / H; e < 16 * (n + 1) / H; e++) mx = fmaxf(mx, st[Q][e]);
          if constexpr (n == H - 1) {
            mx = max_halves(mx);
            mn = fmaxf(m, mx * sc);
          }
        } else {
          constexpr int k = n - H, N = 2 * KD - H;
          constexpr int lo = 16 * k / N, hi = 16 * (k + 1) / N;
#pragma unroll
          for (int e = lo; e < hi; e++) {
            float p = __builtin_amdgcn_exp2f(st[Q][e] * sc - mn);
            ps += p;
            asm volatile("" : "+v"(p), "+v"(ps));  // (here, not where it is used)
            st[Q][e] = p;
          }
          if constexpr (lo < 8 && hi >= 8) {
            pf[Q][0] = acc_to_b(st[Q], 0);
            asm volatile("" : "+v"(pf[Q][0]));
          }
          if constexpr (hi == 16) {
            pf[Q][1] = acc_to_b(st[Q], 1);
            asm volatile("" : "+v"(pf[Q][1]));
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto pv = [&](auto NC) {
      constexpr int n = decltype(NC)::value;
      if constexpr (do_pv) acc[n % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n], pf[P][n / DT], acc[n % DT], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<H>([&](auto NC) {
      pv(NC);
      between(NC);
    });
    wait_dma();  // this wavefront's part of K(u), V(u - 1)
    // and its reads of V(u - 2), a block's softmax ago: behind the barrier V(u) takes their buffer, and a wavefront waits only for its own.
    wait_lgkm0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(rk, Q);
    if constexpr (do_s) {
#pragma unroll
      for (int i = 0; i < KD; i++)
        if (i < KA) kf[i] = fr.template rows<P * B, 0>(i);
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<KD - H>([&](auto NC) {
      constexpr int n = H + decltype(NC)::value;
      pv(std::integral_constant<int, n>{});
      between(std::integral_constant<int, n>{});
    });
    issue(rv, 2 + P);
    __builtin_amdgcn_sched_barrier(0);
    static_for<KD>([&](auto NC) {
      constexpr int n = decltype(NC)::value;
      if constexpr (do_s) {
        if constexpr (n + KA < KD) kf[n + KA] = fr.template rows<P * B, 0>(n + KA);
      }
      if constexpr (do_sm) vf[n] = fr.template cols<(2 + Q) * B, n / DT>(n % DT);
      if constexpr (do_s) {
        if constexpr (n == 0) st[P] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[0], zero16(), 0, 0, 0);
        else st[P] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[n], qf[n], st[P], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      between(std::integral_constant<int, KD + n>{});
    });
    if constexpr (do_sm) {
      if (__any(mn > m)) {  // rescale only when some row's maximum moved
        const float corr = __builtin_amdgcn_exp2f(m - mn);
        l *= corr;
#pragma unroll
        for (int t = 0; t < DT; t++)
#pragma unroll
          for (int e = 0; e < 16; e++) acc[t][e] *= corr;
        m = mn;
      }
      l += ps;
    }
  };
  using Y = std::true_type;
  using N = std::false_type;
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  // The last block has parity 0.  The products of the first full iteration find zeros.
  if (nblk & 1) {
    issue(rk, 0);
    iter(P0{}, Y{}, N{}, N{}, N{});
  } else {
    issue(rk, 1);
    iter(P1{}, Y{}, N{}, N{}, N{});
    iter(P0{}, Y{}, Y{}, N{}, Y{});
  }
  for (int u = 2; u < nblk; u += 2) {
    iter(P1{}, Y{}, Y{}, N{}, Y{});
    iter(P0{}, Y{}, Y{}, N{}, Y{});
  }
  iter(P1{}, N{}, Y{}, Y{}, Y{});
#pragma unroll
  for (int n = 0; n < KD; n++) acc[n % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n], pf[0][n / DT], acc[n % DT], 0, 0, 0);
  wait_dma();
  __syncthreads();
  l += __shfl_xor(l, 32, 64);
  // the odd wavefront of a pair hands its sums over
  f32x4* mine = reinterpret_cast<f32x4*>(&lds[0][0]) + (wave >> 1) * (DT * 4 + 1) * 64 + lane;
  if (kh) {
#pragma unroll
    for (int t = 0; t < DT; t++)
#pragma unroll
      for (int g = 0; g < 4; g++) mine[(t * 4 + g) * 64] = f32x4{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
    mine[DT * 4 * 64] = f32x4{m, l, 0.f, 0.f};
  }
  __syncthreads();
  if (kh) return;
  const f32x4 other = mine[DT * 4 * 64];
  const float mm = fmaxf(m, other[0]), a0 = __builtin_amdgcn_exp2f(m - mm), a1 = __builtin_amdgcn_exp2f(other[0] - mm);
  l = l * a0 + other[1] * a1;
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const f32x4 v = mine[(t * 4 + g) * 64];
#pragma unroll
      for (int r = 0; r < 4; r++) acc[t][4 * g + r] = acc[t][4 * g + r] * a0 + v[r] * a1;
    }
  const float inv = 1.f / l;
  bf16_t* ob = o + int64_t(bi) * S * ldo;
#pragma unroll
  for (int t = 0; t < DT; t++) store_t(ob, ldo, qi, hq * D + t * 32, acc[t], inv, lane, qi < S);
  if (lane < 32 && qi < S) lse[(int64_t(bi) * nq + hq) * S + qi] = (mm + __builtin_amdgcn_logf(l)) * LN2;
}

// ================================================================ backward: dQ
// Same decomposition as the forward.  Per KV block: S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - delta),
// dQ^T += K^T dS^T.
// FORM: forms the row statistics and writes them out; otherwise they are there.
template <int D>
constexpr int dq_lds() { return 4 * Tile<D>::BYTES; }
template <int D, bool FORM>
__device__ __forceinline__ void attn_dq(char* lds_, int qb, int hq, int bi, int nb, const bf16_t* __restrict__ qkv, int64_t ld,
                                        const bf16_t* __restrict__ o, int64_t ld_o, const bf16_t* __restrict__ d_o, int64_t ldo,
                                        const float* __restrict__ lse, float* __restrict__ stats, bf16_t* __restrict__ dqkv, int64_t ldg,
                                        int S, int nq, int nkv, const float* __restrict__ cos_tab, const float* __restrict__ sin_tab) {
  using TL = Tile<D>;
  constexpr int KD = D / 16, DT = D / 32;
  bf16_t* lds = reinterpret_cast<bf16_t*>(lds_);  // [2][K | V][TR * D]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hk = hq / (nq / nkv);
  const bf16_t* base = qkv + int64_t(bi) * S * ld;
  const bf16_t* dob = d_o + int64_t(bi) * S * ldo;
  const int q0 = qb * 128, qw = q0 + wave * 32, qi = qw + (lane & 31);
  const float scale = rsqrtf((float)D), sc = scale * LOG2E;
  const i32x4 rsrc = make_rsrc(base, uint32_t(int64_t(S) * ld * 2));
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MLS_LDS bf16_t*)lds;
  TL tl;
  tl.init(ld, wave, lane);
  auto issue = [&](int blk, bool live) {
    const uint32_t t = lds0 + (blk & 1) * 2 * TL::BYTES;
    tl.dma(rsrc, ld, blk * TR, (nq + hk) * D, t, wave, live);
    tl.dma(rsrc, ld, blk * TR, (nq + nkv + hk) * D, t + TL::BYTES, wave, live);
  };

  bf16x8 qf[KD], dof[KD];
#pragma unroll
  for (int kk = 0; kk < KD; kk++) {
    qf[kk] = gfrag(base, ld, qi, hq * D + kk * 16 + (lane >> 5) * 8, qi < S);
    dof[kk] = gfrag(dob, ldo, qi, hq * D + kk * 16 + (lane >> 5) * 8, qi < S);
  }
  const int64_t si = (int64_t(bi) * nq + hq) * S + qi;
  float L2, dl = 0.f;
  if constexpr (FORM) {
    L2 = qi < S ? lse[si] * LOG2E : 0.f;
    // delta = dO . O of this lane's query row (the two lane halves hold complementary features).  The row statistics are
    // written out as the dK / dV kernel takes them: lse log2(e), then -delta, each [b][n_q][S]
    const bf16_t* ob = o + int64_t(bi) * S * ld_o;
#pragma unroll
    for (int kk = 0; kk < KD; kk++) {
      const bf16x8 of = gfrag(ob, ld_o, qi, hq * D + kk * 16 + (lane >> 5) * 8, qi < S);
#pragma unroll
      for (int e = 0; e < 8; e++) dl += (float)of[e] * (float)dof[kk][e];
    }
    dl += __shfl_xor(dl, 32, 64);
    if (lane < 32 && qi < S) {
      stats[si] = L2;
      stats[int64_t(nb) * nq * S + si] = -dl;
    }
  } else {
    L2 = qi < S ? stats[si] : 0.f;
    dl = qi < S ? -stats[int64_t(nb) * nq * S + si] : 0.f;
  }
  // the compiler's own wait for what was loaded, here and not in the loop, where it would be one for the requests of the next block
#pragma unroll
  for (int kk = 0; kk < KD; kk++) asm volatile("" : "+v"(qf[kk]), "+v"(dof[kk]));
  asm volatile("" : "+v"(L2), "+v"(dl));

  f32x16 acc[DT];
#pragma unroll
  for (int t = 0; t < DT; t++) acc[t] = zero16();

  const int kv_end = min(S, q0 + 128);
  const int nblk = (kv_end + TR - 1) / TR;
  issue(0, true);
  for (int blk = 0; blk < nblk; blk++) {
    const int cur = blk & 1, j0 = blk * TR;
    wait_dma();
    __syncthreads();
    issue(blk + 1, blk + 1 < nblk);
    if (j0 <= qw + 31) {
      const bf16_t* ks = lds + cur * 2 * TR * D;
      const bf16_t* vs = ks + TR * D;
      const bool diag = j0 + TR - 1 > qw;  // some pair of this wave is masked
      // one 32-key sub-block at a time, so that only one S^T / dP^T pair is live
#pragma unroll
      for (int jt = 0; jt < 2; jt++) {
        f32x16 st = zero16(), dp = zero16();
        read_ahead<2 * KD, 3, 1>(
            [&](int i) { return TL::frag_rows((i & 1) ? vs : ks, jt, i >> 1, lane); },
            [&](int i, const bf16x8& f) {
              if (i & 1) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, dof[i >> 1], dp, 0, 0, 0);
              else st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[i >> 1], st, 0, 0, 0);
            });
        // key j = j0 + 32 jt + 4 (lane / 32) + off(e) is masked when j > qi, i.e. off(e) > lim; the mask arithmetic
        // is compiled only into the diagonal-block path
        const int lim = qi - (j0 + jt * 32 + (lane >> 5) * 4);
        auto to_ds = [&](auto MASK) {
#pragma unroll
          for (int e = 0; e < 16; e++) {
            float p = __builtin_amdgcn_exp2f(st[e] * sc - L2);
            if (decltype(MASK)::value && 8 * (e >> 2) + (e & 3) > lim) p = 0.f;
            st[e] = p * (dp[e] - dl);
          }
        };
        if (diag) to_ds(std::true_type{}); else to_ds(std::false_type{});
        const bf16x8 df[2] = {acc_to_b(st, 0), acc_to_b(st, 1)};
        read_ahead<2 * DT, 2, 2>([&](int i) { return TL::frag_cols(ks, i % DT, jt * 2 + i / DT, lane); },
                                 [&](int i, const bf16x8& f) {
                                   acc[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, df[i / DT], acc[i % DT], 0, 0, 0);
                                 });
      }
    }
  }
  wait_dma();
  bf16_t* out = dqkv + int64_t(bi) * S * ldg;
  if (cos_tab) {  // the gradient w.r.t. the rotated q, turned back to the projection's output on the way out
    store_t_unrotate<D>(out, ldg, qi, qi, hq * D, acc, scale, cos_tab, sin_tab, lane, qi < S);
  } else {
#pragma unroll
    for (int t = 0; t < DT; t++) store_t(out, ldg, qi, hq * D + t * 32, acc[t], scale, lane, qi < S);
  }
}

template <int D>
__global__ __launch_bounds__(AT_THREADS, 2) void attn_dq_kernel(const bf16_t* __restrict__ qkv, int64_t ld, const bf16_t* __restrict__ o, int64_t ld_o,
                                                                const bf16_t* __restrict__ d_o, int64_t ldo, const float* __restrict__ lse,
                                                                float* __restrict__ stats, bf16_t* __restrict__ dqkv, int64_t ldg, int S, int nq,
                                                                int nkv, const float* __restrict__ cos_tab, const float* __restrict__ sin_tab) {
  __shared__ __attribute__((aligned(1024))) char lds[dq_lds<D>()];
  attn_dq<D, true>(lds, gridDim.y - 1 - blockIdx.y, blockIdx.x, blockIdx.z, gridDim.z, qkv, ld, o, ld_o, d_o, ldo, lse, stats, dqkv, ldg, S, nq, nkv,
                   cos_tab, sin_tab);
}

// ================================================================ backward: dK and dV
// grid (n_kv * nsplit, kv blocks of 128 KT, b), longest first; wave w owns the 32 KT key rows from j0 + 32 KT w and keeps
// their K and V as B operands.  Loops over the query heads of the group and the 32-row query steps at or below the
// diagonal: S = Q K^T (lane column = key row), dP = dO V^T, dS = P (dP - delta), dV^T += dO^T P, dK^T += Q^T dS.
//
// One kernel for both: apart (S formed twice more, 370 us for 32 heads of 128 at 4096 positions) two workgroups fitted a
// CU; together 272 us.  One wavefront per SIMD with up to 512 registers, software-pipelined: step `it` issues S(it), then
// dP(it) with the exponentials of S(it) in between, then the products dV, dK of step it-1 with dS(it) in between, so that
// no product waits for the vector instructions it depends on.  The instructions of a step are issued in exactly the
// order written.  What bounds it is the issue of that one wavefront: about 330 instructions beside the 64 products of a
// step with KT = 2 (MFMAs busy 52 % of the cycles; the wavefront issues 44 % of its time, waits 31 % for a busy unit and 25 %
// for LDS, the barrier or requests; no bank conflicts), so work was taken out of it: delta is where dP starts from, lse arrives
// scaled, requests move by 32-bit offsets.  A 32-row fragment of Q or dO feeds KT
// products; with KT = 2 V no longer fits the registers beside 256 accumulators and is read from LDS.
// Measured (us, before -> after): 4096 positions, 32 heads of 128: 370 -> 272 (KT = 2); 2048, 16 of 128: 145 -> 63; 4096, 16 of
// 64: 210 -> 95; 4096, 16 heads of 128 over 2 KV heads: 286 -> 157 with the reduction.
// LDS: V of the workgroup's keys if it lives there, a ring of five steps [Q | dO | row statistics].  The one
// barrier of a step lies within S(it): step it+1 has landed for everyone, and the slot of step it-2 is free for it+3
// (its last reads came before the Q fragments that S(it) has waited for, and LDS reads return in order).
// With DS, ds takes dS of every head for the dQ kernel, in bf16 as it enters dK.  Tiles of 32 query rows x 32 keys at or below the
// diagonal, a row of tiles after the other; a tile is 2 KiB as the accumulators hold it: rows 16 h .. 16 h + 15 in its half
// h, 16 bytes per lane = key lane % 32, rows 4 (lane / 32) .. +3 and 8 + 4 (lane / 32) .. +3.
constexpr int DS_TILE = 2048;
__host__ __device__ __forceinline__ int64_t ds_head_bytes(int S) {
  const int64_t n = (S + 31) / 32;
  return n * (n + 1) / 2 * DS_TILE;
}
template <int D, int KT>
constexpr int dkv_lds() { return (KT == 2 ? 4 * 32 * KT * D * 2 : 0) + 5 * (2 * Tile<D, 32>::BYTES + 512); }
// x: KV head and part of its group; kb: key block; bi: sequence, of nb
template <int D, int KT, bool DS>
__device__ __forceinline__ void attn_dkv(char* lds, int x, int kb, int bi, int nb, const bf16_t* __restrict__ qkv, int64_t ld, const bf16_t* __restrict__ d_o, int64_t ldo,
                                         const float* __restrict__ stats, bf16_t* __restrict__ dqkv, int64_t ldg, int S, int nq, int nkv,
                                         int nsplit, float* __restrict__ part, const float* __restrict__ cos_tab,
                                         const float* __restrict__ sin_tab, char* __restrict__ ds) {
  using TS = Tile<D, 32>;
  constexpr int KD = D / 16, DT = D / 32, KR = 32 * KT, SLOTS = 5;
  constexpr bool VL = KT == 2;                               // V fragments from LDS
  static_assert(KT == 1 || D == 128);
  constexpr int STG = 2 * TS::BYTES + 512, V_BYTES = VL ? 4 * KR * D * 2 : 0;
  constexpr int NREQ = 2 * TS::NI + 1;                       // requests of a wavefront per step
  constexpr int NST = DS ? 2 * KT : 0;                       // and stores of dS
  static_assert(dkv_lds<D, KT>() == V_BYTES + SLOTS * STG);    // lds: [V] [slot][Q|dO|lse log2(e)|-delta]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  // nsplit > 1: the query heads of a group are shared out over nsplit workgroups (few KV heads would otherwise
  // leave most CUs idle); each writes its fp32 partial sum to `part`, which gqa_reduce_kernel adds up in order
  const int hk = x / nsplit, sp = x % nsplit;
  const int grp = nq / nkv / nsplit, hq0 = hk * (nq / nkv) + sp * grp;
  const bf16_t* base = qkv + int64_t(bi) * S * ld;
  const bf16_t* dob = d_o + int64_t(bi) * S * ldo;
  const int j0 = kb * 4 * KR, jw = j0 + wave * KR;
  const float scale = rsqrtf((float)D), sc = scale * LOG2E;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MLS_LDS char*)lds;
  const uint32_t ring = lds0 + V_BYTES;

  const int q0 = j0 / 32, nst = (S + 31) / 32 - q0;  // first query step, steps per head
  const int niter = nst * grp;
  TS tq, td;
  tq.init(ld, wave, lane);
  td.init(ldo, wave, lane);
  // The query steps of a head are walked from the last one down to the diagonal: the workgroups of all key blocks of that
  // head (same XCD, started together) then read the same Q / dO rows at about the same time and share them in L2.
  // The next request: byte offsets of its rows behind the three descriptors, moved on by a step or to the next head's last step.
  const i32x4 rs_q = make_rsrc(base, uint32_t(int64_t(S) * ld * 2)), rs_d = make_rsrc(dob, uint32_t(int64_t(S) * ldo * 2));
  // even wavefronts fetch lse log2(e), odd ones -delta (each pair the same values)
  const i32x4 rs_s = make_rsrc(stats + ((wave & 1) * int64_t(nb) * nq + int64_t(bi) * nq + hq0) * S, uint32_t(grp * S) * 4);
  int r_i = nst - 1, r_slot = 0, r_left = niter;
  uint32_t o_q = uint32_t((q0 + r_i) * 64 * ld) + hq0 * D * 2, o_d = uint32_t((q0 + r_i) * 64 * ldo) + hq0 * D * 2, o_s = (q0 + r_i) * 128;
  const uint32_t step_q = uint32_t(64 * ld), step_d = uint32_t(64 * ldo);
  const uint32_t wrap_q = (nst - 1) * step_q + D * 2, wrap_d = (nst - 1) * step_d + D * 2, wrap_s = (nst - 1) * 128 + S * 4;
  const uint32_t dst0 = ring + wave * TS::NI * 1024;
  auto issue_q = [&]() {  // requests beyond the last step are sent as empty
    const uint32_t o = r_left > 0 ? o_q : OOB;
#pragma unroll
    for (int i = 0; i < TS::NI; i++) dma16(rs_q, o + tq.off[i], dst0 + r_slot + i * 1024);
  };
  auto issue_d = [&]() {
    const uint32_t o = r_left > 0 ? o_d : OOB;
#pragma unroll
    for (int i = 0; i < TS::NI; i++) dma16(rs_d, o + td.off[i], dst0 + r_slot + TS::BYTES + i * 1024);
  };
  auto issue_s = [&]() {
    const int rows = r_left > 0 ? S - (q0 + r_i) * 32 : 0;
    dma4(rs_s, lane < rows ? o_s + uint32_t(lane) * 4 : OOB, ring + r_slot + 2 * TS::BYTES + (wave & 1) * 256);
    r_left--;
    r_slot = r_slot == (SLOTS - 1) * STG ? 0 : r_slot + STG;
    const bool wrap = r_i == 0;
    r_i = wrap ? nst - 1 : r_i - 1;
    o_q += wrap ? wrap_q : 0u - step_q;
    o_d += wrap ? wrap_d : 0u - step_d;
    o_s += wrap ? wrap_s : 0u - 128u;
  };

  bf16x8 kf[KT][KD], vf[VL ? 1 : KT][KD];
  if constexpr (VL) {
    const i32x4 src = make_rsrc(base + (nq + nkv + hk) * D + int64_t(jw) * ld, jw < S ? uint32_t(int64_t(S - jw) * ld * 2) : 0u);
#pragma unroll
    for (int q = 0; q < KR * D * 2 / 1024; q++) {
      const int row = q * 4 + (lane >> 4), chunk = (lane & 15) ^ (((row & 3) << 2) | ((row >> 2) & 3));
      dma16(src, uint32_t((int64_t(row) * ld + chunk * 8) * 2), lds0 + wave * KR * D * 2 + q * 1024);
    }
  }
#pragma unroll
  for (int kt = 0; kt < KT; kt++) {
    const int ji = jw + kt * 32 + (lane & 31);
#pragma unroll
    for (int kk = 0; kk < KD; kk++) {
      kf[kt][kk] = gfrag(base, ld, ji, (nq + hk) * D + kk * 16 + half * 8, ji < S);
      if constexpr (!VL) vf[kt][kk] = gfrag(base, ld, ji, (nq + nkv + hk) * D + kk * 16 + half * 8, ji < S);
    }
  }
  for (int i = 0; i < 3; i++) {
    issue_q();
    issue_d();
    issue_s();
  }

  f32x16 dk[KT][DT], dv[KT][DT];
#pragma unroll
  for (int kt = 0; kt < KT; kt++)
#pragma unroll
    for (int t = 0; t < DT; t++) dk[kt][t] = dv[kt][t] = zero16();
  bf16x8 pf[KT][2] = {}, df[KT][2] = {};  // P and dS of the previous step

  // Fragment addresses: the swizzle turns a step along the columns into an XOR, slots are multiples of 256 bytes apart.
  uint32_t ra = ring + toff<D>(lane & 31, half * 8) * 2;                                                           // rows: this step's slot
  uint32_t ca = ring + toff<D>(half * 4 + ((lane & 15) >> 2), ((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;        // columns: the step before
  const uint32_t va = ra - V_BYTES + wave * (VL ? KR * D * 2 : 0);
  uint32_t sa = ring + 2 * TS::BYTES + half * 16;

  // The fragment reads of a step in their order: Q rows; dO rows, each followed by V's if those are in LDS; the columns of dO
  // and Q in turn.  Reads run FA fragments ahead of the MFMAs, over the end of the step into the next one's Q rows.
  constexpr int G = VL ? 1 + KT : 1;
  constexpr int R1 = KD, R2 = R1 + KD * G, R3 = R2 + 4 * DT;
  constexpr int FA = KD < 6 ? KD : 6;
  bf16x8 f[R3 + FA];
  auto read = [&](auto IC) {
    constexpr int i = decltype(IC)::value;
    if constexpr (i < R1) {
      f[i] = *(const MLS_LDS bf16x8*)(ra ^ (i << 5));
    } else if constexpr (i < R2) {
      constexpr int kk = (i - R1) / G, w = (i - R1) % G;
      if constexpr (w == 0) f[i] = *(const MLS_LDS bf16x8*)((ra ^ (kk << 5)) + TS::BYTES);
      else f[i] = *(const MLS_LDS bf16x8*)((va ^ (kk << 5)) + (w - 1) * 32 * D * 2);
    } else if constexpr (i < R3) {
      constexpr int q = (i - R2) / 2, ct = q % DT, o = (((i - R2) & 1) ? 0 : TS::BYTES) + q / DT * 16 * D * 2;
      const s16x4 l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)((ca ^ (ct << 6)) + o));
      const s16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)((ca ^ (ct << 6) ^ 32) + (o + 8 * D * 2)));
      const s16x8 v = {l[0], l[1], l[2], l[3], h[0], h[1], h[2], h[3]};
      f[i] = __builtin_bit_cast(bf16x8, v);
    } else {
      f[i] = *(const MLS_LDS bf16x8*)(ra ^ ((i - R3) << 5));  // the row address has moved on
    }
  };
  // Products that take fragment i (with V in LDS a dP product goes with the V fragment).  S and dP are products in asm that
  // leave their results in VGPRs (the compiler would put them beside dK and dV into AGPRs and copy them back and forth);
  // their first reader stays three products (96 cycles; two would do) behind the last one that wrote them, which the fixed
  // order below sees to: the compiler may move nothing across a product.
  f32x16 st[KT], dp[KT];
  // dP starts from -delta.
  auto mul = [&](f32x16& c, const bf16x8& x, const bf16x8& y, auto ZERO) {
    if constexpr (decltype(ZERO)::value) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(x), "v"(y));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(x), "v"(y));
  };
  auto use = [&](auto IC) {
    constexpr int i = decltype(IC)::value;
    if constexpr (i < R1) {
#pragma unroll
      for (int kt = 0; kt < KT; kt++) mul(st[kt], f[i], kf[kt][i], std::bool_constant<i == 0>{});
    } else if constexpr (i < R2) {
      constexpr int kk = (i - R1) / G, w = (i - R1) % G;
      if constexpr (VL) {
        if constexpr (w > 0) mul(dp[w - 1], f[R1 + kk * G], f[i], std::false_type{});
      } else {
#pragma unroll
        for (int kt = 0; kt < KT; kt++) mul(dp[kt], f[i], vf[kt][kk], std::false_type{});
      }
    } else {
      constexpr int q = (i - R2) / 2;
#pragma unroll
      for (int kt = 0; kt < KT; kt++) {
        if constexpr ((i - R2) & 1) dk[kt][q % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], df[kt][q / DT], dk[kt][q % DT], 0, 0, 0);
        else dv[kt][q % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], pf[kt][q / DT], dv[kt][q % DT], 0, 0, 0);
      }
    }
  };
  // fragments [LO, HI) in exactly this order: the read FA ahead (up to END), the products, vector instructions between(i)
  auto run = [&](auto LO, auto HI, auto END, auto&& between) {
    constexpr int lo = decltype(LO)::value, hi = decltype(HI)::value, end = decltype(END)::value;
    static_for<hi - lo>([&](auto IC) {
      constexpr int i = lo + decltype(IC)::value;
      if constexpr (i + FA < end) read(std::integral_constant<int, i + FA>{});
      use(std::integral_constant<int, i>{});
      __builtin_amdgcn_sched_barrier(0);  // no vector instruction of this group ahead of its products
      between(std::integral_constant<int, i>{});
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto none = [](auto) {};
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, R1>;
  using I2 = std::integral_constant<int, R2>;
  using I3 = std::integral_constant<int, R3>;
  using I4 = std::integral_constant<int, R3 + FA>;

  int slot = 0;
  uint32_t adv = 0;  // from the previous step's slot to this one's
#pragma unroll
  for (int kt = 0; kt < KT; kt++)  // the compiler's own wait for the K (and V) fragments, here and not in the loop
#pragma unroll
    for (int kk = 0; kk < KD; kk++) {
      asm volatile("" : "+v"(kf[kt][kk]));
      if constexpr (!VL) asm volatile("" : "+v"(vf[kt][kk]));
    }
  wait_vmcnt<2 * NREQ>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  // The last `dead` steps of a head have no row that sees a key of this wavefront.  They pass it by: their probabilities are
  // zeros, which would take nothing from a finite row of Q or dO, but make NaN of one with an infinity in it.
  const int dead = min(nst, (jw - j0) / 32), alive = nst - dead;
  for (int hd = 0; hd < grp; hd++) {
    int i0 = (q0 + nst - 1) * 32;  // of this step
    const auto rs_ds = __builtin_amdgcn_make_buffer_rsrc(DS ? ds + (int64_t(bi) * nq + hq0 + hd) * ds_head_bytes(S) : nullptr, 0, DS ? int(ds_head_bytes(S)) : 0, 0x00020000);
    static_for<FA>(read);
    for (int it = 0; it < alive; it++) {
      // ---- S(it)
      constexpr int Q1 = R1 / 4;
      run(I0{}, std::integral_constant<int, Q1>{}, I3{}, none);
      // (the stores of the step before may be on their way too; a head's first step may follow on one without)
      if (DS && it > 0) wait_vmcnt<NREQ + NST>(); else wait_vmcnt<NREQ>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      issue_q();
      run(std::integral_constant<int, Q1>{}, std::integral_constant<int, 2 * Q1>{}, I3{}, none);
      issue_d();
      run(std::integral_constant<int, 2 * Q1>{}, std::integral_constant<int, 3 * Q1>{}, I3{}, none);
      issue_s();
      f32x4 ls[4];  // lse log2(e) of 4 rows each: read one group ahead of use
      ls[0] = *(const MLS_LDS f32x4*)(sa);
#pragma unroll
      for (int kt = 0; kt < KT; kt++) {
        uint32_t da = sa;
        asm volatile("" : "+v"(da));  // read again for each key tile: copies would be vector instructions
#pragma unroll
        for (int g = 0; g < 4; g++) {
          const f32x4 v = *(const MLS_LDS f32x4*)(da + 256 + g * 32);
#pragma unroll
          for (int r = 0; r < 4; r++) dp[kt][g * 4 + r] = v[r];
        }
      }
      run(std::integral_constant<int, 3 * Q1>{}, I1{}, I3{}, none);
      // ---- dP(it); P(it) = exp2(sc S - L2)
      run(I1{}, I2{}, I3{}, [&](auto IC) {
        constexpr int n = R2 - R1, i = decltype(IC)::value - R1, b0 = VL ? 4 : KT == 1 ? 2 : 1;  // three products behind S
        if constexpr (i >= b0) {
          constexpr int lo = (i - b0) * 16 * KT / (n - b0), hi = (i - b0 + 1) * 16 * KT / (n - b0);
          static_for<hi - lo>([&](auto EC) {
            constexpr int x = lo + decltype(EC)::value, g = x / (4 * KT), kt = x / 4 % KT, e = g * 4 + x % 4;
            if constexpr (x % (4 * KT) == 0 && g < 3) ls[g + 1] = *(const MLS_LDS f32x4*)(sa + (g + 1) * 32);
            st[kt][e] = __builtin_amdgcn_exp2f(st[kt][e] * sc - ls[g][x % 4]);
          });
        }
      });
      if (i0 < jw + KR - 1 || i0 + 32 > S) {  // wave-uniform: some pair is masked, or the step runs past the last row
#pragma unroll
        for (int kt = 0; kt < KT; kt++) {
          const int c = jw + kt * 32 + (lane & 31) - i0 - half * 4, z = S - i0 - half * 4;
#pragma unroll
          for (int e = 0; e < 16; e++) {
            const int r = 8 * (e >> 2) + (e & 3);
            if (r < c || r >= z) st[kt][e] = 0.f;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // ---- dV, dK of step it-1; dS(it) = P dP, which has delta taken off
      const uint32_t next = slot == SLOTS - 1 ? 0u - (SLOTS - 1) * STG : STG;
      ra += next;
      run(I2{}, I3{}, I4{}, [&](auto IC) {
        constexpr int n = R3 - R2, i = decltype(IC)::value - R2, b0 = 2;  // three products and more behind dP
        if constexpr (i >= b0) {
          constexpr int lo = (i - b0) * 16 * KT / (n - b0), hi = (i - b0 + 1) * 16 * KT / (n - b0);
          static_for<hi - lo>([&](auto EC) {
            constexpr int x = lo + decltype(EC)::value, g = x / (4 * KT), kt = x / 4 % KT, e = g * 4 + x % 4;
            dp[kt][e] *= st[kt][e];
            if constexpr (e == 7) {  // the products with the previous step's first halves have been issued
              static_assert(i >= n / 2 - 1);
              pf[kt][0] = acc_to_b(st[kt], 0);
              df[kt][0] = acc_to_b(dp[kt], 0);
            }
          });
        }
      });
#pragma unroll
      for (int kt = 0; kt < KT; kt++) {
        pf[kt][1] = acc_to_b(st[kt], 1);
        df[kt][1] = acc_to_b(dp[kt], 1);
      }
      if constexpr (DS) {  // as many stores in every step: those above the diagonal go nowhere
        const int qs = i0 / 32, kt0 = jw / 32;
#pragma unroll
        for (int kt = 0; kt < KT; kt++)
#pragma unroll
          for (int h = 0; h < 2; h++)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, df[kt][h]), rs_ds, kt0 + kt <= qs ? lane * 16 : int(OOB),
                                                   (qs * (qs + 1) / 2 + kt0 + kt) * DS_TILE + h * 1024, 0);
      }
      static_for<FA>([&](auto IC) { f[decltype(IC)::value] = f[R3 + decltype(IC)::value]; });
      ca += adv;  // the columns move on to this step's slot (in a head's first step, which has no predecessor, they were there already)
      sa += next;
      adv = next;
      slot = slot == SLOTS - 1 ? 0 : slot + 1;
      i0 -= 32;
      __builtin_amdgcn_sched_barrier(0);
    }
    // the products of the last step
    static_for<FA>([&](auto IC) { read(std::integral_constant<int, R2 + decltype(IC)::value>{}); });
    run(I2{}, I3{}, I3{}, none);
#pragma unroll
    for (int kt = 0; kt < KT; kt++) pf[kt][0] = pf[kt][1] = df[kt][0] = df[kt][1] = bf16x8{};
    for (int it = 0; it < dead; it++) {
      wait_vmcnt<NREQ>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      issue_q();
      issue_d();
      issue_s();
      const uint32_t next = slot == SLOTS - 1 ? 0u - (SLOTS - 1) * STG : STG;
      ra += next;
      ca += adv;
      sa += next;
      adv = next;
      slot = slot == SLOTS - 1 ? 0 : slot + 1;
    }
    ca += adv;  // to the next head's first step
    adv = 0;
  }
  wait_dma();

#pragma unroll
  for (int kt = 0; kt < KT; kt++) {
    const int ji = jw + kt * 32 + (lane & 31);
    if (nsplit == 1) {
      bf16_t* out = dqkv + int64_t(bi) * S * ldg;
      if (cos_tab) {  // dK is a gradient w.r.t. the rotated k (partial sums are turned back by the reduction)
        store_t_unrotate<D>(out, ldg, ji, ji, (nq + hk) * D, dk[kt], scale, cos_tab, sin_tab, lane, ji < S);
      } else {
#pragma unroll
        for (int t = 0; t < DT; t++) store_t(out, ldg, ji, (nq + hk) * D + t * 32, dk[kt][t], scale, lane, ji < S);
      }
#pragma unroll
      for (int t = 0; t < DT; t++) store_t(out, ldg, ji, (nq + nkv + hk) * D + t * 32, dv[kt][t], 1.f, lane, ji < S);
    } else if (ji < S) {
      // part: [dK | dV][b][n_kv][nsplit][S][D] fp32
      float* out = part + (((int64_t(bi) * nkv + hk) * nsplit + sp) * S + ji) * D;
      const int64_t whole = int64_t(nb) * nkv * nsplit * S * D;
#pragma unroll
      for (int t = 0; t < DT; t++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
          const int c = t * 32 + half * 4 + 8 * g;
          *reinterpret_cast<float4*>(out + c) = make_float4(dk[kt][t][g * 4] * scale, dk[kt][t][g * 4 + 1] * scale,
                                                            dk[kt][t][g * 4 + 2] * scale, dk[kt][t][g * 4 + 3] * scale);
          *reinterpret_cast<float4*>(out + whole + c) =
              make_float4(dv[kt][t][g * 4], dv[kt][t][g * 4 + 1], dv[kt][t][g * 4 + 2], dv[kt][t][g * 4 + 3]);
        }
    }
  }
}

template <int D, int KT>
__global__ __launch_bounds__(AT_THREADS, 1) void attn_dkv_kernel(const bf16_t* __restrict__ qkv, int64_t ld, const bf16_t* __restrict__ d_o,
                                                                 int64_t ldo, const float* __restrict__ stats, bf16_t* __restrict__ dqkv,
                                                                 int64_t ldg, int S, int nq, int nkv, int nsplit, float* __restrict__ part,
                                                                 const float* __restrict__ cos_tab, const float* __restrict__ sin_tab) {
  __shared__ __attribute__((aligned(1024))) char lds[dkv_lds<D, KT>()];
  attn_dkv<D, KT, false>(lds, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z, qkv, ld, d_o, ldo, stats, dqkv, ldg, S, nq, nkv, nsplit, part, cos_tab, sin_tab, nullptr);
}
template <int D, int KT>
__global__ __launch_bounds__(AT_THREADS, 1) void attn_dkv_ds_kernel(const bf16_t* __restrict__ qkv, int64_t ld, const bf16_t* __restrict__ d_o,
                                                                    int64_t ldo, const float* __restrict__ stats, bf16_t* __restrict__ dqkv,
                                                                    int64_t ldg, int S, int nq, int nkv, int nsplit, float* __restrict__ part,
                                                                    const float* __restrict__ cos_tab, const float* __restrict__ sin_tab,
                                                                    char* __restrict__ ds) {
  __shared__ __attribute__((aligned(1024))) char lds[dkv_lds<D, KT>()];
  attn_dkv<D, KT, true>(lds, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z, qkv, ld, d_o, ldo, stats, dqkv, ldg, S, nq, nkv, nsplit, part, cos_tab, sin_tab, ds);
}

// ================================================================ backward: dQ, dK and dV in one launch
// Both kernels above on row statistics that attn_stats_kernel has formed.  Apart, each lasts as long as its longest causal chain while
// the CUs with short ones idle; together the one's short chains run beside the other's long ones.  grid ((n_kv nsplit + n_q) b, blocks of
// 128): rank by rank, the longest first, a rank's key blocks before its query blocks.  Heads of 64 have two workgroups per CU, of 128 one
// (the registers of the dK / dV part).  Whole backward (us, apart or with dQ from dS -> this): 2 x 1000 positions, 16 heads of 64 over 4:
// 51 -> 39; 512, 16 of 64: 28 -> 18; 1024, 16 of 128: 59 -> 40; 2048, 16 of 128: 100 -> 84; 512, 16 of 128: 38.5 -> 27; 2 x 128, 4 of
// 64: 16.3 -> 11.9.  The second half of the ranks in ascending order, so that two workgroups of a CU are long and short: slower (2048 x 16
// of 128 98, 4096 x 16 of 64 155 instead of 147).  With heads of 128 the compiler keeps the results of the dQ part in AGPRs here, which costs
// it 192 copies per 48 products.
template <int D>
__global__ __launch_bounds__(AT_THREADS, D == 64 ? 2 : 1) void attn_bwd_kernel(const bf16_t* __restrict__ qkv, int64_t ld, const bf16_t* __restrict__ d_o,
                                                                               int64_t ldo, float* __restrict__ stats, bf16_t* __restrict__ dqkv,
                                                                               int64_t ldg, int S, int nq, int nkv, int nsplit, int b,
                                                                               float* __restrict__ part, const float* __restrict__ cos_tab,
                                                                               const float* __restrict__ sin_tab) {
  __shared__ __attribute__((aligned(1024))) char lds[dq_lds<D>() > dkv_lds<D, 1>() ? dq_lds<D>() : dkv_lds<D, 1>()];
  const int rank = blockIdx.y, bi = blockIdx.x % b, x = blockIdx.x / b;
  if (x < nkv * nsplit)
    attn_dkv<D, 1, false>(lds, x, rank, bi, b, qkv, ld, d_o, ldo, stats, dqkv, ldg, S, nq, nkv, nsplit, part, cos_tab, sin_tab, nullptr);
  else
    attn_dq<D, false>(lds, gridDim.y - 1 - rank, x - nkv * nsplit, bi, b, qkv, ld, nullptr, 0, d_o, ldo, nullptr, stats, dqkv, ldg, S, nq, nkv, cos_tab, sin_tab);
}

// ================================================================ backward: dQ from the dS of the dK / dV kernel
// The row statistics that the dK / dV kernel takes, when no dQ kernel forms them: lse log2(e), then -(dO . O), each [b][n_q][S].
// grid (n_q, blocks of 64 positions, b).  HBM-bound.
template <int D>
__global__ __launch_bounds__(AT_THREADS) void attn_stats_kernel(const bf16_t* __restrict__ o, int64_t ld_o, const bf16_t* __restrict__ d_o,
                                                                int64_t ldo, const float* __restrict__ lse, float* __restrict__ stats, int S,
                                                                int nq) {
  constexpr int L = D / 8, G = AT_THREADS / L;  // lanes per row, rows at a time
  const int hq = blockIdx.x, bi = blockIdx.z, c = threadIdx.x % L * 8;
  uint4 vo[64 / G], vd[64 / G];
#pragma unroll
  for (int i = 0; i < 64 / G; i++) {
    const int64_t row = int64_t(bi) * S + min(int(blockIdx.y) * 64 + i * G + int(threadIdx.x) / L, S - 1);
    vo[i] = *reinterpret_cast<const uint4*>(o + row * ld_o + hq * D + c);
    vd[i] = *reinterpret_cast<const uint4*>(d_o + row * ldo + hq * D + c);
  }
#pragma unroll
  for (int i = 0; i < 64 / G; i++) {
    const bf16x8 a = __builtin_bit_cast(bf16x8, vo[i]), b = __builtin_bit_cast(bf16x8, vd[i]);
    float dl = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e++) dl += (float)a[e] * (float)b[e];
#pragma unroll
    for (int m = 1; m < L; m <<= 1) dl += __shfl_xor(dl, m, 64);
    const int q = blockIdx.y * 64 + i * G + threadIdx.x / L;
    if (threadIdx.x % L == 0 && q < S) {
      const int64_t si = (int64_t(bi) * nq + hq) * S + q;
      stats[si] = lse[si] * LOG2E;
      stats[int64_t(gridDim.z) * nq * S + si] = -dl;
    }
  }
}

// dQ^T += K^T dS^T over the keys at or below the diagonal.  grid (n_q, q blocks of 128, b), longest first; wave w owns query rows
// q0 + 32 w .. +31 and streams its own row of dS tiles; the K tiles of 64 keys are shared.  HBM-bound, if enough is on its way:
// K comes two deep and dS three deep by LDS-DMA, two workgroups per CU.
template <int D>
__global__ __launch_bounds__(AT_THREADS, 2) void attn_dq_ds_kernel(const bf16_t* __restrict__ qkv, int64_t ld, const char* __restrict__ ds,
                                                                   bf16_t* __restrict__ dqkv, int64_t ldg, int S, int nq, int nkv,
                                                                   const float* __restrict__ cos_tab, const float* __restrict__ sin_tab) {
  using TL = Tile<D>;
  constexpr int DT = D / 32, DSB = 2 * DS_TILE;  // dS of a wavefront per block of 64 keys
  constexpr int NDS = 3, RING = 2 * TL::BYTES;   // dS stages, behind the two of K
  __shared__ __attribute__((aligned(1024))) char lds[RING + NDS * 4 * DSB];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qb = gridDim.y - 1 - blockIdx.y;
  const int hq = blockIdx.x, bi = blockIdx.z, hk = hq / (nq / nkv);
  const bf16_t* base = qkv + int64_t(bi) * S * ld;
  const int q0 = qb * 128, qs = q0 / 32 + wave, qi = qs * 32 + (lane & 31);
  const i32x4 rk = make_rsrc(base, uint32_t(int64_t(S) * ld * 2));
  // this wavefront's row of tiles; what lies beyond the diagonal is out of its range
  const i32x4 rd = make_rsrc(ds + (int64_t(bi) * nq + hq) * ds_head_bytes(S) + int64_t(qs) * (qs + 1) / 2 * DS_TILE,
                             qs * 32 < S ? uint32_t(qs + 1) * DS_TILE : 0u);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MLS_LDS char*)&lds[0];
  TL tl;
  tl.init(ld, wave, lane);
  // LDS keeps the chunks of the second lane half with bit 2 of the key inverted (the transposing reads below)
  const uint32_t src = ((lane & 32) + ((lane & 31) ^ (lane >> 5 << 2))) * 16;
  const int nblk = (min(S, q0 + 128) + TR - 1) / TR;
  auto issue_k = [&](int blk) { tl.dma(rk, ld, blk * TR, (nq + hk) * D, lds0 + (blk & 1) * TL::BYTES, wave, blk < nblk); };
  int ds_slot = 0;  // of the next request
  auto issue_ds = [&](int blk) {
#pragma unroll
    for (int i = 0; i < DSB / 1024; i++)
      dma16(rd, blk < nblk ? blk * DSB + i * 1024 + src : OOB, lds0 + RING + (ds_slot * 4 + wave) * DSB + i * 1024);
    ds_slot = ds_slot == NDS - 1 ? 0 : ds_slot + 1;
  };
  // 16 keys x 32 rows of a tile as an operand: key and row of this lane's share (see Tile::frag_cols)
  const int kr = (lane >> 5) * 4 + ((lane & 15) >> 2), c4 = lane & 3;
  const uint32_t fr = ((lane >> 4) & 1) * 1024 + (((c4 & 1) * 32 + (kr ^ ((c4 & 1) << 2))) * 16) + (c4 >> 1) * 8;
  f32x16 acc[DT];
#pragma unroll
  for (int t = 0; t < DT; t++) acc[t] = zero16();
  issue_ds(0);
  issue_k(0);
  issue_ds(1);
  int at = 0;  // this block's stage of dS
  for (int blk = 0; blk < nblk; blk++) {
    wait_vmcnt<DSB / 1024>();  // all but the dS of the next block
    __syncthreads();
    issue_k(blk + 1);
    issue_ds(blk + 2);
    const bf16_t* ks = reinterpret_cast<const bf16_t*>(lds + (blk & 1) * TL::BYTES);
    const char* dst = lds + RING + (at * 4 + wave) * DSB;
    at = at == NDS - 1 ? 0 : at + 1;
#pragma unroll
    for (int jt = 0; jt < 2; jt++) {
      if (blk * 2 + jt > qs) break;  // (wave-uniform: no row of this wavefront sees a key of the tile)
      bf16x8 df[2];
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const char* a = dst + jt * DS_TILE + fr + k * 256;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)a);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLS_LDS s16x4*)(a + 128));
        const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        df[k] = __builtin_bit_cast(bf16x8, v);
      }
      read_ahead<2 * DT, 3, 2>([&](int i) { return TL::frag_cols(ks, i % DT, jt * 2 + i / DT, lane); },
                               [&](int i, const bf16x8& f) {
                                 acc[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, df[i / DT], acc[i % DT], 0, 0, 0);
                               });
    }
  }
  wait_dma();
  const float scale = rsqrtf((float)D);
  bf16_t* out = dqkv + int64_t(bi) * S * ldg;
  if (cos_tab) {
    store_t_unrotate<D>(out, ldg, qi, qi, hq * D, acc, scale, cos_tab, sin_tab, lane, qi < S);
  } else {
#pragma unroll
    for (int t = 0; t < DT; t++) store_t(out, ldg, qi, hq * D + t * 32, acc[t], scale, lane, qi < S);
  }
}

// dK, dV <- the partial sums of the nsplit workgroups of each KV head, added in ascending order.  A thread owns 8
// features of the first half of a head vector and their 8 partners in the second half, so that dK (a gradient
// w.r.t. the rotated k) can be turned back by the rotary angle when the tables are given.
__global__ __launch_bounds__(256) void gqa_reduce_kernel(const float* __restrict__ part, int nsplit, int b, int S, int D,
                                                         int nq, int nkv, bf16_t* __restrict__ dqkv, int64_t ldg,
                                                         const float* __restrict__ cos_tab,
                                                         const float* __restrict__ sin_tab) {
  const int64_t id = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int d2 = D >> 1, cpr = d2 >> 3;
  const int64_t total = int64_t(2) * b * nkv * S * cpr;
  if (id >= total) return;
  const int c = int(id % cpr) * 8;
  const int64_t row = id / cpr;               // (what, bi, hk, token)
  const int token = int(row % S);
  const int hk = int((row / S) % nkv), bi = int((row / S / nkv) % b), what = int(row / S / nkv / b);
  const float* p = part + ((((int64_t(what) * b + bi) * nkv + hk) * nsplit) * S + token) * D + c;
  float a1[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, a2[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int sp = 0; sp < nsplit; sp++) {
    float v1[8], v2[8];
    load8(p + int64_t(sp) * S * D, v1);
    load8(p + int64_t(sp) * S * D + d2, v2);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      a1[e] += v1[e];
      a2[e] += v2[e];
    }
  }
  if (what == 0 && cos_tab) {
    float cs[8], sn[8];
    load8(cos_tab + int64_t(token) * d2 + c, cs);
    load8(sin_tab + int64_t(token) * d2 + c, sn);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const float g1 = a1[e], g2 = a2[e];
      a1[e] = g1 * cs[e] + g2 * sn[e];
      a2[e] = g2 * cs[e] - g1 * sn[e];
    }
  }
  bf16_t* out = dqkv + (int64_t(bi) * S + token) * ldg + (what ? nq + nkv + hk : nq + hk) * D + c;
  store8(out, a1);
  store8(out + d2, a2);
}

}  // namespace

namespace mls {

// The forward on pairs of wavefronts pays where the longest chain of the other kernel decides, that is up to about one of its workgroups
// (of 128 rows) per CU; with more of them the second load of every key block costs more than the balance gains.  us, other / pairs:
//   d = 128: 160 workgroups 14.9 / 12.7 (512 positions), 240 17.5 / 15.2 (700), 320 45.5 / 34.7 (2048), 384 47.1 / 43.6 (2048) but
//            17.7 / 18.7 (384), 448 49.4 / 47.9 (2048), 512 53.2 / 53.0 (2048), 768 68 / 74 (2048)
//   d = 64:  320 12.0 / 10.0 (600), 384 11.3 / 9.2 (384), 29.5 / 24.1 (2048), 448 14.5 / 13.9 (800), 480 11.8 / 13.1 (384), 512 31.5 / 28.8 (2048)
// Short sequences have short chains: the pairs gain half a microsecond on few workgroups (128 positions 6.8 / 6.5, 300 9.3 / 8.1) and lose one
// on more (192 workgroups of 256 9.9 / 10.6, 256 of 256 10.5 / 11.3), so they stay with the other kernel.
// From 384 positions on, where the pairs' own workgroups (of 64 rows) outnumber their places, or where heads x sequences is no multiple of 8, so
// that the blocks of a head, 8 and 8 more apart, lie on several XCDs and each fetches its keys for itself, on all eight if the number is odd:
//   d = 128, no more pairs than places (512): 41 heads of 448 positions 12.8 / 13.1, 63 of 448 14.3 / 15.7, 43 of 576 16.3 / 17.1 but 54 of 448
//            13.3 / 12.8, 37 of 600 16.5 / 15.9; more: 92 of 384 15.3 / 19.6, 80 of 430 14.9 / 16.9, 62 of 600 20.2 / 22.5 but 64 of 576 20.8 / 16.9;
//            from 832 positions on pairs all the same: 46 of 896 25.4 / 25.5, 42 29.8 / 20.2
//   d = 64:  83 of 400 9.7 / 10.2, 107 of 384 10.0 / 10.8, 74 of 513 11.8 / 12.4 but 96 of 384 9.4 / 9.2, 66 of 513 14.2 / 10.2, 58 of 700 13.8 / 13.6
bool fwd_pairs(int b, int S, int nq, int d) {
  const int64_t heads = int64_t(b) * nq, pairs = heads * ((S + 63) / 64);
  if (S < 384 || heads * ((S + 127) / 128) > (d == 64 ? 384 : 320)) return false;
  const bool own_xcd = heads % 8 == 0;
  if (d == 64) return own_xcd || S >= 640 || pairs <= (S > 512 ? 600 : 576);
  if (S >= 832) return true;
  return pairs <= 512 ? heads % 2 == 0 || heads <= 40 : own_xcd && S > 512;
}

hipError_t attn_fwd_bf16(const void* qkv, int64_t ld_qkv, void* o, int64_t ld_o, float* lse, int b, int S, int nq, int nkv,
                         int d, hipStream_t st) {
  if (b == 0 || S == 0) return hipSuccess;
  if (d != 128 && d != 64) return hipErrorInvalidValue;
  if (fwd_pairs(b, S, nq, d)) {
    auto kern = d == 128 ? attn_fwd_pair_kernel<128> : attn_fwd_pair_kernel<64>;
    hipLaunchKernelGGL(kern, dim3(nq * b, (S + 63) / 64), dim3(AT_THREADS), 0, st, (const bf16_t*)qkv, ld_qkv, (bf16_t*)o, ld_o, lse, S, nq, nkv);
    return hipGetLastError();
  }
  dim3 grid(nq, (S + 127) / 128, b);
  auto kern = d == 128 ? attn_fwd_kernel<128> : attn_fwd_kernel<64>;
  hipLaunchKernelGGL(kern, grid, dim3(AT_THREADS), 0, st, (const bf16_t*)qkv, ld_qkv, (bf16_t*)o, ld_o, lse, S, nq, nkv);
  return hipGetLastError();
}

// dK / dV kernel: key tiles per wavefront, and how many workgroups share the query heads of one KV group.  The smallest
// estimate of max(longest workgroup, share of a CU) in steps of 32 query rows, plus the reduction of partial sums.
// Measured us per step: 1.1 (d = 128, one key tile: 32 heads at 4096 in 292 us), 1.95 (two: 272 us, half the steps),
// 0.75 (d = 64; two tiles were slower: 130 against 95 us for 16 heads at 4096).  Two tiles win once every CU has
// several workgroups, one tile below: 16 heads at 2048 63 against 105 us.  Partial sums of 16.8 million floats: 12 us.
struct DkvPlan { int kt, ns; };
DkvPlan dkv_plan(int b, int S, int nq, int nkv, int d) {
  DkvPlan best{1, 1};
  double least = 1e300;
  const int steps = (S + 31) / 32, grp = nq / nkv;
  for (int kt = 1; kt <= (d == 128 ? 2 : 1); kt++) {
    const int nb = (S + 128 * kt - 1) / (128 * kt);
    const double sum = double(nb) * steps - double(nb) * (nb - 1) / 2 * 4 * kt;  // steps of all key blocks, one head
    for (int ns = 1; ns <= grp; ns++) {
      if (grp % ns) continue;
      const double longest = double(steps) * (grp / ns), share = sum * nq * b / 256;
      double t = (d == 64 ? 0.75 : kt == 1 ? 1.1 : 1.95) * (longest > share ? longest : share);
      if (ns > 1) t += 4 + 0.8e-6 * 2 * b * nkv * double(ns) * S * d;
      if (t < least) least = t, best = {kt, ns};
    }
  }
  return best;
}

// dQ, dK and dV in one launch: up to about as many workgroups of 128 query rows as have a place on the chip at once, beyond which the
// workgroups that follow balance the chip by themselves and the launch costs dQ the second (64: the third) workgroup per CU it has alone.  Whole
// backward, best other / together (us):
//   d = 128: 128 workgroups 32.3 / 25.6 (120 positions), 59 / 40 (1024), 256 100 / 84 (2048), 43.1 / 42.7 (256), 288 90.9 / 89.6 (1500), 320
//            114 / 120 (2048), 512 151 / 161; of one row block 192 28.4 / 29.7, 34.5 / 35.7, 224 36.8 / 38.7
//   d = 64:  320 87 / 64 (2048), 512 101 / 86 (2048), 768 132 / 125 (2048), 26.4 / 20.1 (64), 1024 303 / 280 (4096), 54.4 / 55.9 (128), 2048 295 / 313
//            (2048), 4096 1008 / 1118 (4096)
// Where every query head has KV heads of its own, a launch of short chains is decided by its last round, and heads x sequences that are no
// multiple of 8 spread a head's blocks over the XCDs: fewer workgroups there.
//   d = 128, up to 256 positions: 230 workgroups 31.8 / 33.8 (200 positions), 255 42.6 / 44.4 (384) but 208 (of 104 heads) 35.8 / 33.8 (256)
//   d = 64, one row block: 360 22.0 / 20.7 (100), 402 26.0 / 27.0 (128), 462 15.6 / 18.0 (64), 536 22.0 / 19.2 (64; both take two rounds), 765
//            23.5 / 25.7 (64); two: 500 22.8 / 25.5 (147); up to 448 positions: 662 28.9 / 30.6 (129), 723 43.1 / 45.3 (300), 956 64.6 / 66.3 (448)
//            but 640 (of 160 heads) 45.4 / 38.7 (400)
bool bwd_together(int b, int S, int nq, int nkv, int d) {
  const int64_t heads = int64_t(b) * nq, wgs = heads * ((S + 127) / 128);
  const bool own_xcd = heads % 8 == 0;
  if (nq > nkv) return wgs <= (d == 64 ? (S > 128 ? 1024 : 768) : (S > 128 ? 256 : 128));
  if (d == 128) return wgs <= (S <= 128 ? 128 : own_xcd ? 256 : S <= 256 ? 200 : 250);
  if (S <= 128) return wgs <= 360 || (wgs > 512 && wgs <= (own_xcd ? 700 : 620));
  if (S <= 256 && wgs > 420 && wgs <= 512) return false;
  return wgs <= (S <= 448 && !own_xcd ? 600 : 1024);
}

// dQ from dS as the dK / dV kernel leaves it in memory, instead of a kernel that forms S, P and dP once more: two of its three
// products less, for 2 bytes of dS written and read per score and a launch more.  It pays where the dQ kernel is bound by the chain
// of its few workgroups (about one per CU) and dS stays in the 256 MiB memory-side cache, where a little more than one workgroup per CU
// keeps dQ out of the launch of dK and dV (up to 256: 2048 positions, 16 heads of 128 120 twice, 98.5 once, 83.5 together).  Whole backward,
// dS formed once / in one launch (us): 20 heads of 128 over 4 at 2048 positions 115 / 123, 32 over 8 at 1280 86 / 91; twice / once with more
// workgroups: 32 at 2048 152 / 146 (nothing is left of it in a whole step), 48 at 2048 233 / 236, 32 at 4096 461 / 476.
bool dq_from_ds(int b, int S, int nq, int nkv, int d) {
  return d == 128 && S >= 256 && !bwd_together(b, S, nq, nkv, d) && int64_t(b) * nq * ((S + 127) / 128) <= 320 &&
         ds_head_bytes(S) * nq * b <= int64_t(256) << 20;
}

// partial sums of dK and dV, then dS
size_t part_floats(int b, int S, int nq, int nkv, int d) {
  const int n = dkv_plan(b, S, nq, nkv, d).ns;
  return n > 1 ? (size_t(2) * b * nkv * n * S * d + 255) / 256 * 256 : 0;
}
size_t attn_bwd_scratch_floats(int dt, int b, int S, int nq, int nkv, int d) {
  if (nkv <= 0 || nq % nkv) return 0;
  if (dt != DT_BF16) return attn_bwd_f32_scratch_floats(b, S, nq, nkv, d);
  return part_floats(b, S, nq, nkv, d) + (dq_from_ds(b, S, nq, nkv, d) ? size_t(ds_head_bytes(S)) / 4 * nq * b : 0);
}

hipError_t attn_bwd_bf16(const void* qkv, int64_t ld_qkv, const void* o, int64_t ld_o, const float* lse, const void* d_o,
                         int64_t ld_do, void* dqkv, int64_t ld_dqkv, float* stats, int b, int S, int nq, int nkv, int d,
                         hipStream_t st, float* part, const float* cos_tab, const float* sin_tab) {
  if (b == 0 || S == 0) return hipSuccess;
  if (!cos_tab != !sin_tab) return hipErrorInvalidValue;
  if (d != 128 && d != 64) return hipErrorInvalidValue;
  const DkvPlan pl = dkv_plan(b, S, nq, nkv, d);
  char* ds = part && dq_from_ds(b, S, nq, nkv, d) ? reinterpret_cast<char*>(part + part_floats(b, S, nq, nkv, d)) : nullptr;
  const int ns = part ? pl.ns : 1, kt = ds ? 1 : pl.kt;  // (so few workgroups always get one key tile: their longest chain decides)
  dim3 gq(nq, (S + 127) / 128, b), gk(nkv * ns, (S + 128 * kt - 1) / (128 * kt), b);
  if (bwd_together(b, S, nq, nkv, d)) {
    auto stat = d == 128 ? attn_stats_kernel<128> : attn_stats_kernel<64>;
    auto bwd = d == 128 ? attn_bwd_kernel<128> : attn_bwd_kernel<64>;
    hipLaunchKernelGGL(stat, dim3(nq, (S + 63) / 64, b), dim3(AT_THREADS), 0, st, (const bf16_t*)o, ld_o, (const bf16_t*)d_o, ld_do, lse, stats, S, nq);
    hipLaunchKernelGGL(bwd, dim3((nkv * ns + nq) * b, (S + 127) / 128), dim3(AT_THREADS), 0, st, (const bf16_t*)qkv, ld_qkv, (const bf16_t*)d_o, ld_do, stats,
                       (bf16_t*)dqkv, ld_dqkv, S, nq, nkv, ns, b, part, cos_tab, sin_tab);
  } else if (ds) {
    hipLaunchKernelGGL(attn_stats_kernel<128>, dim3(nq, (S + 63) / 64, b), dim3(AT_THREADS), 0, st, (const bf16_t*)o, ld_o, (const bf16_t*)d_o, ld_do, lse, stats, S, nq);
    hipLaunchKernelGGL((attn_dkv_ds_kernel<128, 1>), gk, dim3(AT_THREADS), 0, st, (const bf16_t*)qkv, ld_qkv, (const bf16_t*)d_o, ld_do, stats,
                       (bf16_t*)dqkv, ld_dqkv, S, nq, nkv, ns, part, cos_tab, sin_tab, ds);
    hipLaunchKernelGGL(attn_dq_ds_kernel<128>, gq, dim3(AT_THREADS), 0, st, (const bf16_t*)qkv, ld_qkv, ds, (bf16_t*)dqkv, ld_dqkv, S, nq, nkv, cos_tab, sin_tab);
  } else {
    auto dq = d == 128 ? attn_dq_kernel<128> : attn_dq_kernel<64>;
    auto dkv = d == 64 ? attn_dkv_kernel<64, 1> : kt == 1 ? attn_dkv_kernel<128, 1> : attn_dkv_kernel<128, 2>;
    hipLaunchKernelGGL(dq, gq, dim3(AT_THREADS), 0, st, (const bf16_t*)qkv, ld_qkv, (const bf16_t*)o, ld_o,
                       (const bf16_t*)d_o, ld_do, lse, stats, (bf16_t*)dqkv, ld_dqkv, S, nq, nkv, cos_tab, sin_tab);
    hipLaunchKernelGGL(dkv, gk, dim3(AT_THREADS), 0, st, (const bf16_t*)qkv, ld_qkv, (const bf16_t*)d_o, ld_do, stats,
                       (bf16_t*)dqkv, ld_dqkv, S, nq, nkv, ns, part, cos_tab, sin_tab);
  }
  if (ns > 1) {
    const int64_t total = int64_t(2) * b * nkv * S * (d >> 4);
    hipLaunchKernelGGL(gqa_reduce_kernel, dim3(unsigned((total + 255) / 256)), dim3(256), 0, st, part, ns, b, S, d, nq, nkv,
                       (bf16_t*)dqkv, ld_dqkv, cos_tab, sin_tab);
  }
  return hipGetLastError();
}

hipError_t attn_fwd(int dt, const void* qkv, int64_t ld_qkv, void* o, int64_t ld_o, float* lse, int b, int S, int nq,
                    int nkv, int d, hipStream_t st) {
  return dt == DT_BF16 ? attn_fwd_bf16(qkv, ld_qkv, o, ld_o, lse, b, S, nq, nkv, d, st)
                       : attn_fwd_f32(qkv, ld_qkv, o, ld_o, lse, b, S, nq, nkv, d, st);
}
hipError_t attn_bwd(int dt, const void* qkv, int64_t ld_qkv, const void* o, int64_t ld_o, const float* lse,
                    const void* d_o, int64_t ld_do, void* dqkv, int64_t ld_dqkv, float* delta, int b, int S, int nq,
                    int nkv, int d, hipStream_t st, float* part, const float* cos_tab, const float* sin_tab) {
  return dt == DT_BF16
             ? attn_bwd_bf16(qkv, ld_qkv, o, ld_o, lse, d_o, ld_do, dqkv, ld_dqkv, delta, b, S, nq, nkv, d, st, part, cos_tab, sin_tab)
             : attn_bwd_f32(qkv, ld_qkv, o, ld_o, lse, d_o, ld_do, dqkv, ld_dqkv, delta, b, S, nq, nkv, d, st, part, cos_tab, sin_tab);
}

}  // namespace mls
