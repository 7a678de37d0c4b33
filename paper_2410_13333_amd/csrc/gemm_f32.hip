// fp32 GEMM of the all-fp32 validation mode, on v_mfma_f32_32x32x2_f32 (full fp32 products and sums).  Same three modes
// and epilogues as the bf16 kernel.
//
// The shapes of this mode are small.  What bounds a launch is the chain of K / 2 dependent MFMAs of an output tile, the number
// of tiles, and what the tiles fetch (the 32x32 ones 10 TB/s in all at 512 x 512 x 2752, which is what the L2 caches give).
// Few tiles: the four wavefronts of a workgroup share ONE 32x32 tile and take every fourth 32-deep piece of the contraction
// each; their partial sums meet in a fixed tree through LDS.  Many: 64x64 tiles, a quadrant per wavefront.
// Pieces come by global_load_lds_dwordx4 (whole lines of both operands, 64-bit addresses: any size and stride) and are read into
// registers one piece ahead of their MFMAs.  A lane's MFMA operand is one row (or column) at one k; the order of the
// contraction is free as long as both operands agree, so the two lane halves take k-values 8g .. 8g+3 and 8g+4 .. 8g+7 and an
// operand stored along k is read 16 bytes at a time.
// The loop is issued in its written order: the LDS reads of the next piece go out between the MFMAs (64 clocks each), requests and what ends
// inside a piece are branches that are the same for all lanes.  With reads first and every lane's address selected anew the matrix cores waited
// some 130 instructions per piece.  us, before -> after, the same bits: 512 x 512 x 2752 21.0 -> 16.9, 96 x 512 x 2048 17.1 -> 12.2,
// 1000 x 4096 x 1024 83 -> 73.5 (114 TFLOP/s; these MFMAs alone reach 131 to 137), weight gradient 1024 x 2752 over 1000 tokens 73 -> 59.  Deeper rings
// (four pieces per wavefront, one workgroup per CU: 1000 x 4096 x 1024 77), three workgroups per CU and tiles dealt out by XCD gave nothing.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int KC = 32;  // contraction depth of one piece: whole 128-byte lines of an operand stored along k

// What becomes of a product: stored (+ R, += ); gate|up, whose SwiGLU is stored besides; q|k|v, whose q and k heads are rotated; dZ of
// the down-projection, which stays in registers, its SwiGLU backward stored.
enum { E_STORE, E_SWIGLU, E_ROPE, E_DSWIGLU };
constexpr bool paired(int epi) { return epi == E_SWIGLU || epi == E_ROPE; }
struct Epilogue {
  float* X;            // Z (E_SWIGLU)
  const float *cos_tab, *sin_tab;
  int64_t ldx;
  int half;            // columns between the two of a pair: ffn, or half a head
  int seq, rot_cols;
};
// Where column r of a tile whose first column is n0 lies in C if its columns come in pairs half apart: eight first ones, then their eight
// partners, so that both of a pair end up in one lane (n0: a multiple of 16, half: of 8).  N: all columns, which the last ones repeat.  GROUPS:
// more than one pair of halves.
struct PairedCol {
  int group, at;  // the pair of halves and the column in its first one
  __device__ __forceinline__ int first(int half) const { return group * 2 * half + at; }
};
template <bool GROUPS>
__device__ __forceinline__ PairedCol paired_col(int n0, int r, int half, int N) {
  const int p = min((n0 + r) >> 4, (N >> 4) - 1), w = half >> 3, group = GROUPS ? p / w : 0;  // p: its eight pairs
  return {group, 8 * (p - group * w) + (r & 7)};
}

__device__ __forceinline__ void dma16g(const float* p, uint32_t lds_byte) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_byte), "v"(p) : "memory");
}

// One operand of a tile of 32 NT rows (of C's rows or columns): element (row, k) at base[row * ld + k] (ALONG_K; K a multiple
// of 8, rows 16-byte aligned) or base[k * ld + row] (rows a multiple of 8).  A piece in LDS:
//   ALONG_K   32 NT rows of 128 bytes, their 16-byte chunks permuted by (row >> 1) & 7
//   else      32 k-rows of 32 NT floats; the two lane halves read rows four apart, which must not share banks: rows of 128 bytes
//             change places with their neighbour where bit 2 of k is set, in rows of 256 bytes the halves do
// A wavefront fetches the pieces at k0, k0 + stride, ... by requests q0 .. q0 + NQ - 1 (of 4 NT).  Their addresses move on by
// additions; only a last piece that is not whole forms them anew, and the first one of another matrix: with SEG the contraction runs on
// through nseg matrices of depth K each (list), every one of which ends with a piece of its own.
// Rows beyond the end repeat the last ones (their results are not stored); so do k-values, and `read` zeroes those.
// EPI, if paired (not ALONG_K): its columns in the order of paired_col.
template <int NT, bool ALONG_K, bool SEG, int EPI = E_STORE>
struct Operand {
  static constexpr int CPR = ALONG_K ? 8 : 8 * NT, RPQ = 64 / CPR;  // chunks per row, rows per request
  static constexpr int NQ = NT == 1 ? 4 : 2;  // requests of a wavefront per piece: all, or its share of the workgroup's
  const float* base;
  int64_t ld, step;
  int row0, rows, K, k0, stride, q0, half;
  const float* at[NQ];
  const float* const* list = nullptr;
  int nseg = 1, seg = 0;
  __device__ __forceinline__ const float* place(int i, int lane, int k0_) const {
    const int s = (q0 + i) * RPQ + lane / CPR, c = lane % CPR;
    if (ALONG_K) return base + int64_t(min(row0 + s, rows - 1)) * ld + min(k0_ + 4 * (c ^ ((s >> 1) & 7)), K - 4);
    const int k = NT == 1 ? s ^ ((s >> 2) & 1) : s, col = 4 * (NT == 1 ? c : c ^ (((s >> 2) & 1) << 3));
    const float* at_k = base + int64_t(min(k0_ + k, K - 1)) * ld;
    if constexpr (paired(EPI)) return at_k + (paired_col<EPI == E_ROPE>(row0, col, half, rows).first(half) + ((col >> 3) & 1) * half);
    else return at_k + min(row0 + col, rows - 4);
  }
  __device__ __forceinline__ Operand(const float* base_, int64_t ld_, int row0_, int rows_, int K_, int k0_, int stride_, int q0_, int lane, int half_ = 8)
      : base(base_), ld(ld_), step(ALONG_K ? stride_ : stride_ * ld_), row0(row0_), rows(rows_), K(K_), k0(k0_), stride(stride_), q0(q0_), half(half_) {
#pragma unroll
    for (int i = 0; i < NQ; i++) at[i] = place(i, lane, k0);
  }
  // the next piece into LDS byte lds on (SEG: beyond the last matrix some piece of it)
  __device__ __forceinline__ void request(int lane, uint32_t lds) {
    if constexpr (SEG) {
      const int span = (K + KC - 1) / KC * KC;
      if (k0 >= span) {
        for (; k0 >= span; seg++) k0 -= span;
        base = list[min(seg, nseg - 1)];
#pragma unroll
        for (int i = 0; i < NQ; i++) at[i] = place(i, lane, k0);
      }
    }
    if (k0 + KC <= K) {
#pragma unroll
      for (int i = 0; i < NQ; i++) dma16g(at[i], lds + (q0 + i) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < NQ; i++) dma16g(place(i, lane, min(k0, K - 1)), lds + (q0 + i) * 1024);
    }
#pragma unroll
    for (int i = 0; i < NQ; i++) at[i] += step;
    k0 += stride;
  }
  // k-values 8 G + 4 hf .. + 3 of rows 32 t + l32 of the piece at p
  template <int G>
  __device__ __forceinline__ static void read(const float* p, int t, int l32, int hf, float (&f)[KC / 2]) {
    const int k = 8 * G + 4 * hf;
    if (ALONG_K) {
      const float4 v = *reinterpret_cast<const float4*>(p + (t * 32 + l32) * 32 + (((2 * G + hf) ^ ((l32 >> 1) & 7)) << 2));
      f[4 * G] = v.x; f[4 * G + 1] = v.y; f[4 * G + 2] = v.z; f[4 * G + 3] = v.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; j++) f[4 * G + j] = NT == 1 ? p[((k + j) ^ hf) * 32 + l32] : p[(k + j) * 64 + ((t ^ hf) * 32 + l32)];
    }
  }
  // left: k-values of the piece that exist
  __device__ __forceinline__ static void cut(int hf, int left, float (&f)[KC / 2]) {
#pragma unroll
    for (int e = 0; e < KC / 2; e++) f[e] = 8 * (e / 4) + 4 * hf + e % 4 < left ? f[e] : 0.f;
  }
};

// ---- the results of a 32x32 MFMA tile whose lane holds 4 consecutive columns of row l32 four times, 8 apart
template <int EPI>
__device__ __forceinline__ void store_tile(const f32x16& acc, float* C, const float* R, int row, int col0, int M, int N, int64_t ldc,
                                           int64_t ldr, int add, int hf, const Epilogue& ep) {
  if (row >= M) return;
  auto at4 = [](float* p) { return reinterpret_cast<float4*>(p); };
  auto get4 = [](const float* p, float (&v)[4]) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  };
  if constexpr (paired(EPI)) {
#pragma unroll
    for (int g = 0; g < 4; g += 2) {
      if (col0 + 8 * g >= N) continue;  // N is a multiple of 16 here
      const PairedCol pc = paired_col<EPI == E_ROPE>(col0, 8 * g + 4 * hf, ep.half, N);
      const int first = pc.first(ep.half);
      float a[4], b[4];
#pragma unroll
      for (int e = 0; e < 4; e++) a[e] = acc[4 * g + e], b[e] = acc[4 * g + 4 + e];
      float* c = C + int64_t(row) * ldc + first;
      if constexpr (EPI == E_SWIGLU) {
        float z[4];
#pragma unroll
        for (int e = 0; e < 4; e++) z[e] = a[e] * sigmoidf_(a[e]) * b[e];
        *at4(ep.X + int64_t(row) * ep.ldx + first) = make_float4(z[0], z[1], z[2], z[3]);
      } else if (first < ep.rot_cols) {
        const int64_t t = int64_t(row % ep.seq) * ep.half + pc.at;
        float cs[4], sn[4];
        get4(ep.cos_tab + t, cs);
        get4(ep.sin_tab + t, sn);
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const float u = a[e], v = b[e];
          a[e] = u * cs[e] - v * sn[e];
          b[e] = u * sn[e] + v * cs[e];
        }
      }
      *at4(c) = make_float4(a[0], a[1], a[2], a[3]);
      *at4(c + ep.half) = make_float4(b[0], b[1], b[2], b[3]);
    }
    return;
  }
  float gate[4][4], up[4][4];
  if constexpr (EPI == E_DSWIGLU)
#pragma unroll
    for (int g = 0; g < 4; g++) {  // all on their way together
      const float* p = R + int64_t(row) * ldr + min(col0 + 8 * g + 4 * hf, N - 4);
      get4(p, gate[g]);
      get4(p + ep.half, up[g]);
    }
#pragma unroll
  for (int g = 0; g < 4; g++) {
    const int col = col0 + 8 * g + 4 * hf;  // N is a multiple of 8: groups of four are whole
    if (col >= N) continue;
    float* c = C + int64_t(row) * ldc + col;
    if constexpr (EPI == E_DSWIGLU) {
      float dg[4], du[4];
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const float d = acc[4 * g + e], sg = sigmoidf_(gate[g][e]);
        dg[e] = d * up[g][e] * sg * (1.f + gate[g][e] * (1.f - sg));
        du[e] = d * gate[g][e] * sg;
      }
      *at4(c) = make_float4(dg[0], dg[1], dg[2], dg[3]);
      *at4(c + ep.half) = make_float4(du[0], du[1], du[2], du[3]);
      continue;
    }
    float o[4] = {0.f, 0.f, 0.f, 0.f};
    if (add) get4(c, o);
    else if (R) get4(R + int64_t(row) * ldr + col, o);
    *at4(c) = make_float4(acc[4 * g] + o[0], acc[4 * g + 1] + o[1], acc[4 * g + 2] + o[2], acc[4 * g + 3] + o[3]);
  }
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int e = 0; e < 16; e++) z[e] = 0.f;
  return z;
}
__device__ __forceinline__ f32x16 add16(const f32x16& a, const f32x16& b) {
  f32x16 c;
#pragma unroll
  for (int e = 0; e < 16; e++) c[e] = a[e] + b[e];
  return c;
}

// The products of one piece, in this order: two MFMAs, `between` (waits, the requests of a piece to come), the others with the LDS reads of the
// next piece (eight groups, read(0) .. read(7)) in their shadow.  Operands swapped: a lane ends up with 4 consecutive columns of one row of C.
template <class Between, class Read>
__device__ __forceinline__ void products(f32x16& c, const float (&a)[KC / 2], const float (&b)[KC / 2], Between&& between, Read&& read) {
  static_for<KC / 2>([&](auto Q) {
    constexpr int q = decltype(Q)::value;
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(b[q], a[q], c, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (q == 1) between();
    if constexpr (q >= 2 && q < 10) read(std::integral_constant<int, q - 2>{});
    __builtin_amdgcn_sched_barrier(0);
  });
}

// A(m, k): AK ? A[m*lda + k] : A[k*lda + m]; B(k, n): BK ? B[n*ldb + k] : B[k*ldb + n].  add: C += instead of C =.
// SEG: A and B are the first of nseg matrices each.  Every matrix has sums of its own, which are added up: one chain through all of them would
// round on the growing sum at every product (weight gradients of three micro-batches up to 1.25 times as far from the exact ones).
struct Source {
  const float *A, *B;
  int M, N, K;
  int64_t lda, ldb;
  const float *const *a, *const *b;
  int nseg;
};
// Few tiles: one workgroup per 32x32 tile of C, wavefront w takes pieces w, w + 4, ... through NS stages of its own.
template <bool AK, bool BK, bool SEG, int NS, int EPI>
__device__ __forceinline__ void tile32(float* smem, const Source& s, int m0, int n0, float* C, const float* R, int64_t ldc, int64_t ldr, int add,
                                       const Epilogue& ep) {
  const int M = s.M, N = s.N, K = s.K;
  constexpr int STAGE = 2 * 32 * KC, NREQ = 8;
  using OA = Operand<1, AK, SEG>;
  using OB = Operand<1, BK, SEG, EPI>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, hf = lane >> 5;
  OA oa(s.A, s.lda, m0, M, K, wave * KC, 4 * KC, 0, lane);
  OB ob(s.B, s.ldb, n0, N, K, wave * KC, 4 * KC, 0, lane, ep.half);
  if constexpr (SEG) oa.list = s.a, ob.list = s.b, oa.nseg = ob.nseg = s.nseg;
  const float* mine = smem + wave * NS * STAGE;
  const uint32_t lds = (uint32_t)(uintptr_t)(MLS_LDS float*)(smem) + wave * NS * STAGE * 4;
  auto request = [&](int stage) {
    const uint32_t at = lds + stage * STAGE * 4;
    oa.request(lane, at);
    ob.request(lane, at + STAGE * 2);
  };
  f32x16 acc = zero16(), total = zero16();
  const int each = (K + KC - 1) / KC, pieces = SEG ? each * s.nseg : each;
  const int n = (pieces - wave + 3) / 4;  // of this wavefront (0 if there are fewer than four)
  int in_seg = SEG ? wave % each : 0;     // this piece's place in its matrix
  float a[2][KC / 2], b[2][KC / 2];
  auto read = [&](auto I, int stage, int set) {
    constexpr int i = decltype(I)::value;
    const float* st = mine + stage * STAGE;
    if constexpr (i % 2 == 0) OA::template read<i / 2>(st, 0, l32, hf, a[set]);
    else OB::template read<i / 2>(st + STAGE / 2, 0, l32, hf, b[set]);
  };
  auto cut = [&](int p, int set) {
    const int left = !SEG ? K - (p * 4 + wave) * KC : K % KC ? K - (p * 4 + wave) % each * KC : KC;
    if (left < KC) {
      OA::cut(hf, left, a[set]);
      OB::cut(hf, left, b[set]);
    }
  };
  if (n > 0) {
#pragma unroll
    for (int p = 0; p < NS; p++)
      if (p < n) request(p);
    if (n >= NS) wait_vmcnt<(NS - 1) * NREQ>(); else wait_vmcnt<0>();
    static_for<8>([&](auto I) { read(I, 0, 0); });
    wait_lgkm0();
    cut(0, 0);
  }
  auto step = [&](int p, auto STAGE_OF_P) {  // the products of piece p; piece p + 1 is read meanwhile, p + NS requested into its stage
    constexpr int stage = decltype(STAGE_OF_P)::value, set = stage & 1;
    products(acc, a[set], b[set],
             [&] {
               wait_lgkm0();
               if (p + NS < n) {
                 request(stage);
                 wait_vmcnt<(NS - 1) * NREQ>();
               } else {
                 wait_vmcnt<0>();
               }
             },
             [&](auto I) { read(I, (stage + 1) % NS, set ^ 1); });  // (after the last piece: not used)
    cut(p + 1, set ^ 1);
    if constexpr (SEG) {
      in_seg += 4;
      if (in_seg >= each) {
        in_seg %= each;
        total = add16(total, acc);
        acc = zero16();
      }
    }
  };
  for (int p = 0; p < n; p += NS)
    static_for<NS>([&](auto I) {
      if (p + decltype(I)::value < n) step(p + decltype(I)::value, I);
    });
  wait_lgkm0();
  if constexpr (SEG) acc = add16(total, acc);  // (the wavefront's last piece may not be the end of its matrix)
  // wavefronts 2, 3 -> 0, 1; then 1 -> 0
  float(*part)[16][64] = reinterpret_cast<float(*)[16][64]>(smem);
  __syncthreads();
#pragma unroll
  for (int half = 2; half > 0; half >>= 1) {
    if (wave >= half && wave < 2 * half)
#pragma unroll
      for (int e = 0; e < 16; e++) part[wave - half][e][lane] = acc[e];
    __syncthreads();
    if (wave < half)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[e] += part[wave][e][lane];
    __syncthreads();
  }
  if (wave == 0) store_tile<EPI>(acc, C, R, m0 + l32, n0, M, N, ldc, ldr, add, hf, ep);
}

// Many tiles: one workgroup per 64x64 tile, a quadrant for each wavefront, pieces of both operands shared in a ring of four
// stages.  Four accumulators take every fourth piece each and are added like the sums of the four wavefronts above: same bits.
template <bool AK, bool BK, bool SEG, int EPI>
__device__ __forceinline__ void tile64(float* smem, const Source& s, int m0, int n0, float* C, const float* R, int64_t ldc, int64_t ldr, int add,
                                       const Epilogue& ep) {
  const int M = s.M, N = s.N, K = s.K;
  constexpr int STAGE = 2 * 64 * KC, NS = 4, NREQ = 4;
  using OA = Operand<2, AK, SEG>;
  using OB = Operand<2, BK, SEG, EPI>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, hf = lane >> 5;
  const int wm = wave & 1, wn = wave >> 1;
  OA oa(s.A, s.lda, m0, M, K, 0, KC, 2 * wave, lane);
  OB ob(s.B, s.ldb, n0, N, K, 0, KC, 2 * wave, lane, ep.half);
  if constexpr (SEG) oa.list = s.a, ob.list = s.b, oa.nseg = ob.nseg = s.nseg;
  const uint32_t lds = (uint32_t)(uintptr_t)(MLS_LDS float*)(smem);
  const int each = (K + KC - 1) / KC, pieces = SEG ? each * s.nseg : each;
  auto request = [&](int stage) {  // (beyond the last piece: its last k-value, so that the counts of the waits hold)
    const uint32_t at = lds + stage * STAGE * 4;
    oa.request(lane, at);
    ob.request(lane, at + STAGE * 2);
  };
  f32x16 acc[4] = {zero16(), zero16(), zero16(), zero16()}, total = zero16();
  auto sum = [&] { return add16(add16(acc[0], acc[2]), add16(acc[1], acc[3])); };
  int in_seg = 0;  // this piece's place in its matrix
  if (pieces > 0) {
    float a[2][KC / 2], b[2][KC / 2];
    auto read = [&](auto I, int stage, int set) {
      constexpr int i = decltype(I)::value;
      const float* st = smem + stage * STAGE;
      if constexpr (i % 2 == 0) OA::template read<i / 2>(st, wm, l32, hf, a[set]);
      else OB::template read<i / 2>(st + STAGE / 2, wn, l32, hf, b[set]);
    };
    auto cut = [&](int p, int set) {
      const int left = !SEG ? K - p * KC : K % KC ? K - p % each * KC : KC;
      if (left < KC) {
        OA::cut(hf, left, a[set]);
        OB::cut(hf, left, b[set]);
      }
    };
    auto sync = [&]() {  // the next piece is there for everyone, and everyone has read the one before it
      wait_lgkm0();
      wait_vmcnt<(NS - 2) * NREQ>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
#pragma unroll
    for (int p = 0; p < NS - 1; p++) request(p);
    sync();
    request(NS - 1);
    static_for<8>([&](auto I) { read(I, 0, 0); });
    wait_lgkm0();
    cut(0, 0);
    auto step = [&](int p, auto I) {  // the products of piece p, while piece p + 1 is read (after the last one: not used)
      constexpr int i = decltype(I)::value, set = i & 1;
      products(acc[i], a[set], b[set],
               [&] {
                 sync();
                 request(i);
               },
               [&](auto J) { read(J, (i + 1) % NS, set ^ 1); });
      cut(p + 1, set ^ 1);
      if constexpr (SEG) {
        if (++in_seg == each) {
          in_seg = 0;
          total = add16(total, sum());
          acc[0] = acc[1] = acc[2] = acc[3] = zero16();
        }
      }
    };
    for (int p = 0; p < pieces; p += 4)
      static_for<4>([&](auto I) {
        if (p + decltype(I)::value < pieces) step(p + decltype(I)::value, I);
      });
    wait_vmcnt<0>();
  }
  if constexpr (!SEG) total = sum();
  store_tile<EPI>(total, C, R, m0 + wm * 32 + l32, n0 + wn * 32, M, N, ldc, ldr, add, hf, ep);
}

template <bool AK, bool BK, bool LARGE, int EPI>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B, float* C, const float* R,
                                                          int M, int N, int K, int64_t lda, int64_t ldb, int64_t ldc, int64_t ldr, int add, Epilogue ep) {
  extern __shared__ __attribute__((aligned(1024))) float smem[];
  const Source s = {A, B, M, N, K, lda, ldb, nullptr, nullptr, 1};
  if constexpr (LARGE) tile64<AK, BK, false, EPI>(smem, s, blockIdx.y * 64, blockIdx.x * 64, C, R, ldc, ldr, add, ep);
  else tile32<AK, BK, false, 2, EPI>(smem, s, blockIdx.y * 32, blockIdx.x * 32, C, R, ldc, ldr, add, ep);
}

// The weight gradients of a layer over all micro-batches of a call: C (+)= sum_i A_i^T B_i for each problem of a list, all over matrices of
// the same depth, in one launch.  A launch for each of them and each micro-batch left most of the chip idle between its few tiles' chains
// (weight gradients of a call, us, as events around the launches: hidden 512, ffn 1376, 2 x 512 tokens 142 -> 95; 768, 2048, 3 x 1152 652 -> 424;
// 192, 600, 2 x 384 72 -> 21).  The micro-batches' sums are added up in registers, as the launches added them up in C.
constexpr int MAX_SEGS = 16, MAX_GROUP = 4;
struct TnGroup {
  int nseg, n, K, add;
  struct {
    const float *a[MAX_SEGS], *b[MAX_SEGS];
    float* C;
    int64_t lda, ldb, ldc;
    int M, N, tiles_n, tile0;
  } p[MAX_GROUP];
  mls::Colsum cs;  // the last cs.wgs workgroups add columns up instead
};
template <bool LARGE>
__global__ __launch_bounds__(256, 2) void gemm_f32_tn_group_kernel(TnGroup g) {
  extern __shared__ __attribute__((aligned(1024))) float smem[];
  const int tiles = gridDim.x - g.cs.wgs, t = blockIdx.x;
  if (t >= tiles) {
    colsum_block(g.cs, t - tiles, smem);
    return;
  }
  int i = 0;
  while (i + 1 < g.n && t >= g.p[i + 1].tile0) i++;
  const auto& p = g.p[i];
  const int at = t - p.tile0, m = at / p.tiles_n, n = at - m * p.tiles_n;
  const Source s = {p.a[0], p.b[0], p.M, p.N, g.K, p.lda, p.ldb, p.a, p.b, g.nseg};
  if constexpr (LARGE) tile64<false, false, true, E_STORE>(smem, s, m * 64, n * 64, p.C, nullptr, p.ldc, 0, g.add, Epilogue{});
  else tile32<false, false, true, 2, E_STORE>(smem, s, m * 32, n * 32, p.C, nullptr, p.ldc, 0, g.add, Epilogue{});
}

constexpr int LDS = 4 * 2 * 2 * 32 * KC * 4;  // of every form

template <bool AK, bool BK, int EPI = E_STORE>
hipError_t launch_f32(const float* A, const float* B, float* C, const float* R, int M, int N, int K, int64_t lda, int64_t ldb,
                      int64_t ldc, int64_t ldr, int add, hipStream_t st, const Epilogue& ep = {}) {
  const bool large = mls::gemm_f32_large(M, N, K);
  auto kern = large ? gemm_f32_kernel<AK, BK, true, EPI> : gemm_f32_kernel<AK, BK, false, EPI>;
  static std::atomic<uint64_t> lds_raised[2] = {{0}, {0}};
  if (hipError_t e = mls::raise_lds_limit(reinterpret_cast<const void*>(kern), LDS, lds_raised[large])) return e;
  const int t = large ? 64 : 32;
  hipLaunchKernelGGL(kern, dim3((N + t - 1) / t, (M + t - 1) / t), dim3(256), LDS, st, A, B, C, R, M, N, K, lda, ldb, ldc, ldr, add, ep);
  return hipGetLastError();
}

}  // namespace

namespace mls {

// The 64x64 tiles read half as much per product, one to a CU (a second one shares its matrix cores); the 32x32 ones are four times as many, two of
// them on a CU at a time, and their wavefronts take every fourth piece.  Microseconds as rounds times a tile's chain, fitted to both tile
// sizes at 1 609 shapes (48 to 3000 rows, 64 to 4400 columns, contractions of 64 to 5000); the fullest CU counts more than the average one.  The
// choice is on average 0.3 % slower than the faster of the two.  us, 32x32 / 64x64: 1000 x 4096 x 1024 (1024 large tiles) 92 / 74, 512 x 2752 x 512
// (344) 23.0 / 22.4, 288 x 4096 x 4672 (320) 120 / 156, 1152 x 1024 x 768 (288) 24.7 / 29.0, 1024 x 1024 (256, 1024 small) over 64 8.3 / 5.6, over
// 512 15.7 / 12.4, over 2752 59 / 49, 1152 x 768 (216, 864) over 4096 83 / 70, 1024 x 704 (176, 704) over 768 19.4 / 17.2, over 1376 25.3 / 26.5, 768 x 768
// (144, 576) over 256 9.2 / 8.1, over 512 12.3 / 12.0, 512 x 1024 (128, 512) over 256 6.2 / 8.3, 512 x 512 x 2752 (64, 256) 16.9 / 47.6.
bool gemm_f32_large(int M, int N, int K) {
  auto up = [](int64_t v, int64_t t) { return (v + t - 1) / t; };
  const int64_t big = up(M, 64) * up(N, 64), small = up(M, 32) * up(N, 32), pieces = up(K, KC);
  const double load = 0.8 * double(up(small, 256)) + 0.2 * std::max(1.0, double(small) / 256);
  return 2 + 0.54 * double(pieces * up(big, 256)) < (0.72 * double(up(pieces, 4)) + 0.9) * load;
}

// M, N and row strides multiples of 8, operands 16-byte aligned (as every entry point checks); K a multiple of 8 in the
// NN and NT forms, any length in the TN form (a weight gradient contracts over the tokens).  overwrite (TN): C = instead of +=
hipError_t gemm_f32(int mode, const void* A, const void* B, void* C, const void* R, int M, int N, int K, int64_t lda,
                    int64_t ldb, int64_t ldc, int64_t ldr, hipStream_t st, bool overwrite) {
  if (M == 0 || N == 0) return hipSuccess;
  const float *a = (const float*)A, *b = (const float*)B, *r = (const float*)R;
  float* c = (float*)C;
  switch (mode) {
    case GEMM_NN: return launch_f32<true, false>(a, b, c, r, M, N, K, lda, ldb, ldc, ldr, 0, st);
    case GEMM_NT: return launch_f32<true, true>(a, b, c, r, M, N, K, lda, ldb, ldc, ldr, 0, st);
    case GEMM_TN: return launch_f32<false, false>(a, b, c, nullptr, M, N, K, lda, ldb, ldc, ldr, overwrite ? 0 : 1, st);
    default: return hipErrorInvalidValue;
  }
}

// A launch less than the product and an elementwise kernel after it, and no second pass over its results.  With the rotation back in the
// attention backward's stores, a step: hidden 512, ffn 1376, 2 micro-batches of 2 x 256 tokens (eight launches less) 411 -> 394 us; 768, 2048,
// 3 x 1152 1832 -> 1795; 256, 512, 100 tokens 104 -> 97.  The same arithmetic on the same values.
hipError_t gemm_f32_swiglu(const void* A, const void* W, void* GU, void* Z, int M, int f, int K, int64_t lda, int64_t ldw, int64_t ldgu,
                           int64_t ldz, hipStream_t st) {
  if (M == 0 || f == 0) return hipSuccess;
  if (f % 8) return hipErrorInvalidValue;
  const Epilogue ep = {(float*)Z, nullptr, nullptr, ldz, f, 0, 0};
  return launch_f32<true, false, E_SWIGLU>((const float*)A, (const float*)W, (float*)GU, nullptr, M, 2 * f, K, lda, ldw, ldgu, 0, 0, st, ep);
}
hipError_t gemm_f32_rope(const void* A, const void* W, void* C, int M, int N, int K, int64_t lda, int64_t ldw, int64_t ldc, const float* cos_tab,
                         const float* sin_tab, int seq, int rot_cols, int head_dim, hipStream_t st) {
  if (M == 0 || N == 0) return hipSuccess;
  if (head_dim < 16 || head_dim % 16 || N % head_dim || rot_cols % head_dim || seq < 1) return hipErrorInvalidValue;
  const Epilogue ep = {nullptr, cos_tab, sin_tab, 0, head_dim / 2, seq, rot_cols};
  return launch_f32<true, false, E_ROPE>((const float*)A, (const float*)W, (float*)C, nullptr, M, N, K, lda, ldw, ldc, 0, 0, st, ep);
}
hipError_t gemm_f32_dswiglu(const void* dY, const void* W, const void* GU, void* DGU, int M, int f, int K, int64_t lda, int64_t ldw,
                            int64_t ldgu, int64_t lddgu, hipStream_t st) {
  if (M == 0 || f == 0) return hipSuccess;
  const Epilogue ep = {nullptr, nullptr, nullptr, 0, f, 0, 0};
  return launch_f32<true, true, E_DSWIGLU>((const float*)dY, (const float*)W, (float*)DGU, (const float*)GU, M, f, K, lda, ldw, lddgu, ldgu, 0, st, ep);
}

// The 64x64 tiles where all problems together have 320 of them and more (us, 32x32 / 64x64, events around the launch: hidden 512, ffn 1376 over 48
// tokens 35 / 19, 768 / 2048 over 3 x 1152 409 / 353, 708 tiles over 2 x 512 82 / 83; 156 over 2 x 384 18 / 23).
static int64_t tn_group_tiles(const TnProduct* p, int n, int t) {
  int64_t tiles = 0;
  for (int i = 0; i < n; i++) tiles += int64_t((p[i].M + t - 1) / t) * ((p[i].N + t - 1) / t);
  return tiles;
}
int gemm_f32_tn_group_tile(const TnProduct* p, int n) { return tn_group_tiles(p, n, 64) >= 320 ? 64 : 32; }

hipError_t gemm_f32_tn_group(const TnProduct* p, int n, int nseg, int kseg, hipStream_t st, bool overwrite, const Colsum& cs) {
  if (nseg == 0 || kseg == 0) return hipSuccess;
  if (n < 1 || n > MAX_GROUP || nseg > MAX_SEGS) return hipErrorInvalidValue;
  TnGroup g = {};
  auto up = [](int v, int t) { return int64_t((v + t - 1) / t); };
  const int t = gemm_f32_tn_group_tile(p, n);
  const bool large = t == 64;
  if (tn_group_tiles(p, n, t) + cs.wgs >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  g.nseg = nseg;
  g.K = kseg;
  g.add = overwrite ? 0 : 1;
  g.cs = cs;
  int64_t at = 0;
  for (int i = 0; i < n; i++) {
    if (p[i].M == 0 || p[i].N == 0) continue;
    auto& q = g.p[g.n++];
    for (int j = 0; j < nseg; j++) {
      q.a[j] = (const float*)p[i].A[j];
      q.b[j] = (const float*)p[i].B[j];
    }
    q.C = (float*)p[i].C;
    q.lda = p[i].lda; q.ldb = p[i].ldb; q.ldc = p[i].ldc;
    q.M = p[i].M; q.N = p[i].N;
    q.tiles_n = int(up(p[i].N, t));
    q.tile0 = int(at);
    at += up(p[i].M, t) * q.tiles_n;
  }
  if (g.n == 0) return hipSuccess;
  auto kern = large ? gemm_f32_tn_group_kernel<true> : gemm_f32_tn_group_kernel<false>;
  static std::atomic<uint64_t> lds_raised[2] = {{0}, {0}};
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), LDS, lds_raised[large])) return e;
  hipLaunchKernelGGL(kern, dim3(unsigned(at + cs.wgs)), dim3(256), LDS, st, g);
  return hipGetLastError();
}

}  // namespace mls
