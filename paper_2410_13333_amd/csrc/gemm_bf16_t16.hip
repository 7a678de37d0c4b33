// bf16 GEMM on v_mfma_f32_16x16x32_bf16 for everything that whole rounds of 256x256 tiles (gemm_bf16_m16.hip) do not
// suit: the columns left over, problems with fewer tiles than CUs, and fused forms whose contraction ends inside its
// pair of k-tiles.  Smaller tiles of the same design, 4 wavefronts per workgroup:
//   256x128   half the work per workgroup
//   128x128   a quarter
//   128x64    an eighth
//   64x64     small problems: what bounds them is the chain of one tile, so as many tiles as possible
// (for both of the last two 64x128 where the epilogue needs a whole head or a gate/up pair inside one wavefront)
//
// Main loop: k-tiles are 64 deep (128 bytes of a [row][k] operand's row: whole cache lines), NS stages in LDS filled by
// buffer_load_dwordx4 ... lds.  A k-tile is two steps of one MFMA's depth, whose fragments live in two register sets:
//   first half   MFMAs of step 0, the LDS reads of step 1 in between;
//   wait for this wavefront's share of tile t+1, one workgroup barrier: tile t is read, tile t+1 is there;
//   second half  MFMAs of step 1, the LDS reads of tile t+1's step 0 and the requests for tile t+NS (into tile t's stage)
//                in between.
// So no MFMA waits for LDS, there is one barrier per 64 of depth, and a tile is requested NS - 1/2 iterations before it is
// read.  As in the 256x256 kernel the MFMAs, reads and requests are volatile asm in their issue order.  The contraction
// may end inside a k-tile: lanes whose 16-byte chunk (or k-row) lies beyond the end request out of range and get zeros.
//
// What bounds them: at full chips the data moved per product (a 256x128 tile pulls 1.5 times the bytes per FLOP of a 256x256
// one from L2, about 13 TB/s in all at every size here) and, with it, the power limit: 256x128 runs 1 060 .. 1 130 TFLOP/s
// on N(0,1) operands and 1 450 on zeros (2048 x 4096 x 11008), 128x128 1 000 .. 1 080.  On a few workgroups the chain of a
// k-tile (0.21 us at 64x64).  The tiles they replace ran on v_mfma_f32_32x32x16 with plain two-stage (256x128) or
// three-stage (128x128) pipelines: 822 TFLOP/s in the 2048-token 7B layer (256x128), 10 us instead of 4.3 .. 7.8 on a
// 256-token layer's products (128x128).
//
// LDS map of a stage: the A tile, then the B tile.  [row][64 k]: 128-byte rows, the eight 16-byte chunks permuted by
// (row >> 1) & 7.  [k][col]: rows of the tile's width, XOR swizzled (swz_kcol); both on the global-address side, both
// free of bank conflicts for the reads.
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int BK = 64;
constexpr int MAX_SEGS = 16;

enum { E_BF16 = 0, E_F32 = 1, E_SWIGLU = 2, E_ROPE = 3, E_DSWIGLU = 4 };

// The segmented form runs a list of problems in one launch (the weight gradients of a layer, whose tiles alone would each
// leave most of a last round empty): all over the same pieces, each with operands and a result of its own.
struct SegProblem {
  const bf16_t* a[MAX_SEGS];
  const bf16_t* b[MAX_SEGS];
  void* C;
  int64_t lda, ldb, ldc;
  uint32_t a_bytes, b_bytes;
  int M, N, col0, xf, tiles_m, tile0;  // tile0: its first tile in the launch
};
struct SegArgs {
  int nseg, n;
  SegProblem p[mls::MAX_T16_GROUP];
  mls::Colsum cs;  // the last cs.wgs workgroups add columns up instead
};
struct NoSegs {};
struct RopeArgs {
  const float* cos_tab;
  const float* sin_tab;
  int seq, rot_cols, head_dim;
};

// [k][col] tiles of CB 16-byte chunks per k-row: XOR applied to the chunk index of k-row kr.  A transposing 8-byte read
// takes, per group of 16 lanes, 32 bytes from each of k-rows kr0 .. kr0+3, and 32 lanes (two groups, k-rows 8 apart) go
// through the 64 banks (256 bytes) together: the eight 32-byte pieces must lie in eight different places of a bank round.
// Rows of 256 bytes or more: bits 2, 3 from kr & 3, bit 1 from bit 3 of kr; rows of 128 bytes alternate between the
// halves of a round by themselves, the rest comes from bits 1 and 3 of kr.
template <int CB>
__device__ __forceinline__ constexpr int swz_kcol(int kr) {
  return CB >= 16 ? ((kr & 3) << 2) | (((kr >> 3) & 1) << 1) : (((kr >> 1) & 1) << 2) | (((kr >> 3) & 1) << 1);
}

// Wavefront tile: (16 WTM) x (16 WTN); WGM x (4 / WGM) wavefronts.
template <int WTM, int WTN, int WGM, bool ATR, bool BTR, int EPI, bool SEG, int NS>
struct Cfg {
  static constexpr int WGN = 4 / WGM, BM = 16 * WTM * WGM, BN = 16 * WTN * WGN;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES, LDS = NS * STAGE;
  static constexpr int NQA = BM / 32, NQB = BN / 32;  // requests per wavefront and k-tile
  // workgroups a CU can hold by LDS (of 160 KiB); registers follow
  static constexpr int PER_CU = LDS > 80 * 1024 ? 1 : LDS > 53 * 1024 ? 2 : 3;
};

template <int WTM, int WTN, int WGM, bool ATR, bool BTR, int EPI, bool SEG, int NS, bool SPLIT>
__global__ __launch_bounds__(256, (Cfg<WTM, WTN, WGM, ATR, BTR, EPI, SEG, NS>::PER_CU)) void gemm_t16_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, void* __restrict__ C_, const bf16_t* __restrict__ R, int M_,
    int N_, int K, int64_t lda_, int64_t ldb_, int64_t ldc_, int64_t ldr, uint32_t a_bytes_, uint32_t b_bytes_, int tiles_m_,
    int col0_, void* __restrict__ Xv, int64_t ldx, int xf_, std::conditional_t<SEG, SegArgs, NoSegs> segs, RopeArgs rope, SplitArgs split) {
  using G = Cfg<WTM, WTN, WGM, ATR, BTR, EPI, SEG, NS>;
  constexpr int BM = G::BM, BN = G::BN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  // tile of this workgroup: each XCD gets a contiguous run of tiles, walked in groups of about 1024 rows, N fastest
  int nwg = gridDim.x;
  const int pid = blockIdx.x;
  if constexpr (SEG) {
    nwg -= segs.cs.wgs;
    if (pid >= nwg) {
      colsum_block(segs.cs, pid - nwg, reinterpret_cast<float*>(smem));
      return;
    }
  }
  const int xcd = pid & 7, q8 = nwg >> 3, rem = nwg & 7;
  int tile = xcd * q8 + (xcd < rem ? xcd : rem) + (pid >> 3);
  // the problem it belongs to
  void* Cv = C_;
  int M = M_, N = N_, tiles_m = tiles_m_, tiles = nwg, col0 = col0_, xf = xf_, pr = 0;
  int64_t lda = lda_, ldb = ldb_, ldc = ldc_;
  uint32_t a_bytes = a_bytes_, b_bytes = b_bytes_;
  int part = 0;  // its share of the contraction
  if constexpr (SPLIT) {
    tiles = nwg / split.parts;
    part = tile / tiles;
    tile -= part * tiles;
  }
  if constexpr (SEG) {
    while (pr + 1 < segs.n && tile >= segs.p[pr + 1].tile0) pr++;
    const SegProblem& p = segs.p[pr];
    Cv = p.C;
    M = p.M; N = p.N; tiles_m = p.tiles_m; col0 = p.col0; xf = p.xf;
    lda = p.lda; ldb = p.ldb; ldc = p.ldc;
    a_bytes = p.a_bytes; b_bytes = p.b_bytes;
    tiles = (pr + 1 < segs.n ? segs.p[pr + 1].tile0 : nwg) - p.tile0;
    tile -= p.tile0;
  }
  auto piece_a = [&](int i) { if constexpr (SEG) return segs.p[pr].a[i]; else return A; };
  auto piece_b = [&](int i) { if constexpr (SEG) return segs.p[pr].b[i]; else return B; };
  int nseg = 1;
  if constexpr (SEG) nseg = segs.nseg;
  const int gm = min(1024 / BM, tiles_m);
  const int per_group = gm * (tiles / tiles_m), grp = tile / per_group, first_m = grp * gm;
  const int gsz = min(tiles_m - first_m, gm), in_grp = tile - grp * per_group;
  const int m0 = (first_m + in_grp % gsz) * BM, n0 = (in_grp / gsz) * BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave % WGM) * (16 * WTM), wn = (wave / WGM) * (16 * WTN);
  const int l16 = lane & 15, g4 = lane >> 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MLS_LDS unsigned char*)smem;

  // ---- requests: fixed per-lane byte offsets, the k-tile enters as a scalar.  klim: contraction indices of the tile that
  // exist (BK except for the last tile of a piece).
  constexpr int NQA = G::NQA, NQB = G::NQB, NREQ = NQA + NQB;
  constexpr int CA = BM / 8, CB = BN / 8;  // 16-byte chunks per k-row of a [k][col] tile
  uint32_t goa[NQA], gob[NQB];
  auto set_offsets = [&](int klim) {
#pragma unroll
    for (int i = 0; i < NQA; i++) {
      const int q = wave * NQA + i;
      if (ATR) {
        const int kr = q * (64 / CA) + lane / CA, c = (lane % CA) ^ swz_kcol<CA>(kr);
        goa[i] = m0 + c * 8 < M && kr < klim ? uint32_t((int64_t(kr) * lda + m0 + c * 8) * 2) : OOB;
      } else {
        const int r = q * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
        goa[i] = m0 + r < M && c * 8 < klim ? uint32_t((int64_t(m0 + r) * lda + c * 8) * 2) : OOB;
      }
    }
#pragma unroll
    for (int i = 0; i < NQB; i++) {
      const int q = wave * NQB + i;
      if (BTR) {
        const int kr = q * (64 / CB) + lane / CB, c = (lane % CB) ^ swz_kcol<CB>(kr);
        gob[i] = n0 + c * 8 < N && kr < klim ? uint32_t((int64_t(kr) * ldb + n0 + c * 8) * 2) : OOB;
      } else {
        const int r = q * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
        gob[i] = n0 + r < N && c * 8 < klim ? uint32_t((int64_t(n0 + r) * ldb + c * 8) * 2) : OOB;
      }
    }
  };
  const int tps = (K + BK - 1) / BK, krem = K - (tps - 1) * BK;  // k-tiles per piece, depth of the last one
  int kt0 = 0, nk = nseg * tps;
  if constexpr (SPLIT) {
    kt0 = int(int64_t(tps) * part / split.parts);
    nk = int(int64_t(tps) * (part + 1) / split.parts) - kt0;
  }
  const uint32_t ka = ATR ? uint32_t(lda * (BK * 2)) : BK * 2, kb = BTR ? uint32_t(ldb * (BK * 2)) : BK * 2;
  const i32x4 dead_a = make_rsrc(piece_a(0), 0), dead_b = make_rsrc(piece_b(0), 0);
  i32x4 ra = make_rsrc(piece_a(0), a_bytes), rb = make_rsrc(piece_b(0), b_bytes);
  int rq_tile = 0, rq_seg = 0, rq_in = kt0;  // request cursor: next k-tile, its piece and its index inside the piece
  set_offsets(kt0 == tps - 1 ? krem : BK);
  auto request = [&](uint32_t stage, auto DC) {  // request D of this wavefront for the cursor's k-tile
    constexpr int d = decltype(DC)::value;
    const bool live = rq_tile < nk;
    if constexpr (d < NQA) dma16s(live ? ra : dead_a, goa[d], uint32_t(rq_in) * ka, lds0 + stage + (wave * NQA + d) * 1024);
    else dma16s(live ? rb : dead_b, gob[d - NQA], uint32_t(rq_in) * kb, lds0 + stage + G::A_BYTES + (wave * NQB + d - NQA) * 1024);
  };
  auto advance = [&]() {
    rq_tile++;
    rq_in++;
    if (SEG && rq_in == tps) {
      rq_in = 0;
      rq_seg++;
      const int i = rq_seg < nseg ? rq_seg : nseg - 1;
      ra = make_rsrc(piece_a(i), a_bytes);
      rb = make_rsrc(piece_b(i), b_bytes);
      if (krem < BK && tps > 1) set_offsets(BK);
    }
    if (krem < BK && tps > 1 && rq_in == tps - 1) set_offsets(krem);
  };

  // ---- fragment addresses inside stage 0: for a [row][64 k] operand one per step (the permutation turns the step into an
  // XOR), fragment i at +2048 i; for a [k][col] operand one per fragment, the step at +32 k-rows
  constexpr int NAA = ATR ? WTM : 2, NBA = BTR ? WTN : 2;
  uint32_t fa_b[NAA], fb_b[NBA];
#pragma unroll
  for (int i = 0; i < NAA; i++) {
    const int kr = g4 * 8 + (l16 >> 2), col = wm + i * 16 + (l16 & 3) * 4;
    fa_b[i] = lds0 + (ATR ? kr * (BM * 2) + (((col >> 3) ^ swz_kcol<CA>(kr)) << 4) + (col & 7) * 2
                          : (wm + l16) * 128 + (((i * 4 + g4) ^ ((l16 >> 1) & 7)) << 4));
  }
#pragma unroll
  for (int j = 0; j < NBA; j++) {
    const int kr = g4 * 8 + (l16 >> 2), col = wn + j * 16 + (l16 & 3) * 4;
    fb_b[j] = lds0 + G::A_BYTES + (BTR ? kr * (BN * 2) + (((col >> 3) ^ swz_kcol<CB>(kr)) << 4) + (col & 7) * 2
                                       : (wn + l16) * 128 + (((j * 4 + g4) ^ ((l16 >> 1) & 7)) << 4));
  }
  i32x4 fa[2][WTM], fb[2][WTN];
  // LDS read n (A fragments first) of step ST of the tile in `stage` into fragment set ST
  auto rd = [&](auto STC, auto NC, uint32_t stage) {
    constexpr int st = decltype(STC)::value, n = decltype(NC)::value;
    if constexpr (n < WTM) {
      if constexpr (ATR) lds_read16_tr<st * 32 * BM * 2, BM * 2>(fa[st][n], fa_b[n] + stage);
      else lds_read16<n * 2048>(fa[st][n], fa_b[st] + stage);
    } else {
      if constexpr (BTR) lds_read16_tr<st * 32 * BN * 2, BN * 2>(fb[st][n - WTM], fb_b[n - WTM] + stage);
      else lds_read16<(n - WTM) * 2048>(fb[st][n - WTM], fb_b[st] + stage);
    }
  };
  f32x4 c[WTM][WTN];
#pragma unroll
  for (int i = 0; i < WTM; i++)
#pragma unroll
    for (int j = 0; j < WTN; j++) c[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  constexpr int NM = WTM * WTN, NR = WTM + WTN;
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  // prologue: tiles 0 .. NS-1 requested, step 0 of tile 0 read
#pragma unroll
  for (int s = 0; s < NS; s++) {
    static_for<NREQ>([&](auto DC) { request(s * G::STAGE, DC); });
    advance();
  }
  wait_vmcnt<(NS - 1) * NREQ>();
  __builtin_amdgcn_s_barrier();
  static_for<NR>([&](auto NC) { rd(S0{}, NC, 0); });
  wait_lgkm0();

  uint32_t cur = 0;
  for (int t = 0; t < nk; t++) {
    const uint32_t nxt = cur == (NS - 1) * G::STAGE ? 0 : cur + G::STAGE;
    // first half: the reads go out over the first three quarters of the MFMAs
    static_for<NM>([&](auto MC) {
      constexpr int m = decltype(MC)::value, span = NM * 3 / 4 > 0 ? NM * 3 / 4 : 1;
      mfma16(c[m / WTN][m % WTN], fb[0][m % WTN], fa[0][m / WTN]);
      static_for<NR>([&](auto RC) {
        if constexpr (decltype(RC)::value * span / NR == m) rd(S1{}, RC, cur);
      });
    });
    wait_lgkm0();                      // this wavefront's reads of tile t are back
    wait_vmcnt<(NS - 2) * NREQ>();     // its share of tile t+1 has landed
    __builtin_amdgcn_s_barrier();
    // second half: the reads of tile t+1 over its first part; the requests for tile t+NS into the stage just freed are
    // spread over all of it (as a burst in either part they cost 5 to 8 %)
    static_for<NM>([&](auto MC) {
      constexpr int m = decltype(MC)::value, span = NM / 2 > 0 ? NM / 2 : 1;
      mfma16(c[m / WTN][m % WTN], fb[1][m % WTN], fa[1][m / WTN]);
      static_for<NR>([&](auto RC) {
        if constexpr (decltype(RC)::value * span / NR == m) rd(S0{}, RC, nxt);
      });
      static_for<NREQ>([&](auto DC) {
        if constexpr (decltype(DC)::value * NM / NREQ == m) request(cur, DC);
      });
    });
    // the fragments must have arrived before anything but the issue order above: what follows branches, and the compiler,
    // to which a read's result is there at once, may move registers around a branch
    wait_lgkm0();
    advance();
    // the compiler does not see MFMAs written as asm and inserts no wait states behind them: whatever it places at the
    // loop exit must find the last result written
    asm volatile("s_nop 15" ::: "memory");
    cur = nxt;
  }
  wait_vmcnt<0>();
  __syncthreads();

  if constexpr (SPLIT) {
    if (!join_parts<WTM, WTN>(split, tile, part, c, reinterpret_cast<uint32_t*>(smem))) return;
    __syncthreads();  // (the epilogue writes where the ticket was)
  }

  // ---- epilogue.  Lane l holds, of MFMA tile (i, j): C[row 16 i + l%16][cols 16 j + 4 (l/16) .. +3].
  const int64_t crow0 = m0 + wm, ccol0 = n0 + wn;
  if constexpr (EPI == E_F32) {
    // (ldx != 0 in this mode: store, do not accumulate)
    f32_results<WTM, WTN>(reinterpret_cast<float*>(Cv), ldc, int(crow0), M, int(ccol0), N, col0, xf, ldx == 0, c, lane, smem + wave * (1024 * WTN));
  } else if constexpr (EPI == E_DSWIGLU) {
    // The product is the gradient w.r.t. silu(gate) * up; C gets the gradients w.r.t. both, in the interleaved order of R = gate | up.  Each
    // block of 16 rows passes through fp32 staging so that a lane has eight neighbouring columns: whole 64-byte pieces of gates and ups.
    // All gates and ups are on their way before the first block is needed.  The product is rounded to bf16 first: the bits of the two
    // kernels that run where 256x256 tiles take part.
    constexpr int CH = 4 * WTN, C8 = 2 * WTN, RPI = 64 / C8, NP = 16 / RPI;  // 4-column chunks and 8-column pieces per row, rows per pass, passes
    unsigned char* ws = smem + wave * (1024 * WTN);
    bf16_t* C = reinterpret_cast<bf16_t*>(Cv);
    const int c8 = lane % C8, r0 = lane / C8, n = int(ccol0) + c8 * 8;
    const int64_t at = ((n >> 5) << 6) + (n & 31);  // of the gates; their ups 32 columns further on
    uint4 g[WTM][NP], u[WTM][NP];
#pragma unroll
    for (int i = 0; i < WTM; i++)
#pragma unroll
      for (int q = 0; q < NP; q++) {
        const int64_t row = crow0 + i * 16 + q * RPI + r0;
        g[i][q] = u[i][q] = make_uint4(0, 0, 0, 0);
        if (row < M && n < N) {
          g[i][q] = *reinterpret_cast<const uint4*>(R + row * ldr + at);
          u[i][q] = *reinterpret_cast<const uint4*>(R + row * ldr + at + 32);
        }
      }
#pragma unroll
    for (int i = 0; i < WTM; i++) {
#pragma unroll
      for (int j = 0; j < WTN; j++) *reinterpret_cast<f32x4*>(ws + l16 * (CH * 16) + (((j * 4 + g4) ^ (l16 & (CH - 1))) << 4)) = c[i][j];
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < NP; q++) {
        const int r = q * RPI + r0;
        const int64_t row = crow0 + i * 16 + r;
        const f32x4 lo = *reinterpret_cast<const f32x4*>(ws + r * (CH * 16) + (((2 * c8) ^ (r & (CH - 1))) << 4));
        const f32x4 hi = *reinterpret_cast<const f32x4*>(ws + r * (CH * 16) + (((2 * c8 + 1) ^ (r & (CH - 1))) << 4));
        float gv[8], uv[8], og[8], ou[8];
        load8(reinterpret_cast<const bf16_t*>(&g[i][q]), gv);
        load8(reinterpret_cast<const bf16_t*>(&u[i][q]), uv);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float d = round_bf16(e < 4 ? lo[e] : hi[e - 4]), s = sigmoidf_(gv[e]);
          og[e] = d * uv[e] * s * (1.f + gv[e] * (1.f - s));
          ou[e] = d * gv[e] * s;
        }
        if (row < M && n < N) {
          store8(C + row * ldc + at, og);
          store8(C + row * ldc + at + 32, ou);
        }
      }
      wave_lds_sync();
    }
  } else {
    // bf16 output through a per-wavefront staging area (16 rows x 16 WTN columns, 16-byte chunks XOR-swizzled by row) so
    // that the stores move whole rows.  The fused forms work on the fp32 accumulators first:
    //   E_ROPE    a head lies inside the wavefront's columns: both values of a rotary pair (i, i + head_dim/2) sit in
    //             the same lane, head_dim/32 MFMA tiles apart: rotate, then round once;
    //   E_SWIGLU  columns come as 32 gates, their 32 ups, ...: the up of a gate sits two MFMA tiles to the right in
    //             the same lane; C gets both, X[row][f] their product silu(gate) * up formed in fp32.
    constexpr int CH = 2 * WTN, RPI = 64 / CH;  // chunks per row, rows per store instruction
    unsigned char* ws = smem + wave * (16 * CH * 16 * 2);
    unsigned char* wz = ws + 16 * CH * 16;
    bf16_t* C = reinterpret_cast<bf16_t*>(Cv);
    // columns of this wavefront that are rotated: whole heads (v, behind them, is not)
    const int rot = EPI == E_ROPE ? rope.rot_cols - (col0 + int(ccol0)) : 0;
#pragma unroll
    for (int i = 0; i < WTM; i++) {
      const int64_t row = crow0 + i * 16 + l16;
      float v[WTN][4];
#pragma unroll
      for (int j = 0; j < WTN; j++)
#pragma unroll
        for (int e = 0; e < 4; e++) v[j][e] = c[i][j][e];
      if constexpr (EPI == E_BF16) {
        if (R) {
#pragma unroll
          for (int j = 0; j < WTN; j++) {
            const int col = int(ccol0) + j * 16 + g4 * 4;
            if (row < M && col < N) {
              float r4[4];
              load4(R + row * ldr + col0 + col, r4);
              v[j][0] += r4[0]; v[j][1] += r4[1]; v[j][2] += r4[2]; v[j][3] += r4[3];
            }
          }
        }
      }
      if constexpr (EPI == E_ROPE) {
        // TP = MFMA tiles between the halves of a pair
        auto rotate = [&](auto TPC) {
          constexpr int TP = decltype(TPC)::value;
          const int64_t pos = row < M ? row % rope.seq : 0;
          const float* ct = rope.cos_tab + pos * (16 * TP) + g4 * 4;
          const float* sn = rope.sin_tab + pos * (16 * TP) + g4 * 4;
#pragma unroll
          for (int p = 0; p < TP; p++) {
            const float4 c4 = *reinterpret_cast<const float4*>(ct + 16 * p), s4 = *reinterpret_cast<const float4*>(sn + 16 * p);
            const float cc[4] = {c4.x, c4.y, c4.z, c4.w}, ss[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
            for (int j = p; j + TP < WTN; j += 2 * TP)
#pragma unroll
              for (int e = 0; e < 4 && 16 * j < rot; e++) {
                const float u1 = v[j][e], u2 = v[j + TP][e];
                v[j][e] = u1 * cc[e] - u2 * ss[e];
                v[j + TP][e] = u1 * ss[e] + u2 * cc[e];
              }
          }
        };
        if (rot > 0) {
          if (rope.head_dim == 128) rotate(std::integral_constant<int, 4>{}); else rotate(std::integral_constant<int, 2>{});
        }
      }
#pragma unroll
      for (int j = 0; j < WTN; j++) {
        uint2 o;
        o.x = pack_bf16x2(v[j][0], v[j][1]);
        o.y = pack_bf16x2(v[j][2], v[j][3]);
        const int ch = j * 2 + (g4 >> 1);
        *reinterpret_cast<uint2*>(ws + l16 * (CH * 16) + ((ch ^ (l16 & (CH - 1))) << 4) + (g4 & 1) * 8) = o;
      }
      if constexpr (EPI == E_SWIGLU) {
        // gate tiles 4n, 4n+1 with their ups 4n+2, 4n+3 -> product tiles 2n, 2n+1
#pragma unroll
        for (int zb = 0; zb < WTN / 2; zb++) {
          const int jg = (zb >> 1) * 4 + (zb & 1), ju = jg + 2;
          float z[4];
#pragma unroll
          for (int e = 0; e < 4; e++) z[e] = v[jg][e] * sigmoidf_(v[jg][e]) * v[ju][e];
          uint2 o;
          o.x = pack_bf16x2(z[0], z[1]);
          o.y = pack_bf16x2(z[2], z[3]);
          const int ch = zb * 2 + (g4 >> 1);
          *reinterpret_cast<uint2*>(wz + l16 * (CH * 8) + ((ch ^ (l16 & (CH / 2 - 1))) << 4) + (g4 & 1) * 8) = o;
        }
      }
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < 16 / RPI; q++) {
        const int rr = q * RPI + lane / CH, chk = lane % CH;
        const uint4 o = *reinterpret_cast<const uint4*>(ws + rr * (CH * 16) + ((chk ^ (rr & (CH - 1))) << 4));
        const int64_t grow = crow0 + i * 16 + rr;
        const int gcol = int(ccol0) + chk * 8;
        if (grow < M && gcol < N) *reinterpret_cast<uint4*>(C + grow * ldc + col0 + gcol) = o;
      }
      if constexpr (EPI == E_SWIGLU) {
        bf16_t* X = reinterpret_cast<bf16_t*>(Xv);
        constexpr int ZCH = CH / 2, ZRPI = 64 / ZCH;
#pragma unroll
        for (int q = 0; q < (16 + ZRPI - 1) / ZRPI; q++) {
          const int rr = q * ZRPI + lane / ZCH, chk = lane % ZCH;
          if (rr < 16) {
            const uint4 o = *reinterpret_cast<const uint4*>(wz + rr * (CH * 8) + ((chk ^ (rr & (ZCH - 1))) << 4));
            const int64_t grow = crow0 + i * 16 + rr;
            const int gcol = int(ccol0) + (chk >> 2) * 64 + (chk & 3) * 8;  // the gate column of this chunk's first product
            const int zcol = ((col0 + int(ccol0)) >> 1) + chk * 8;       // its place among the f products
            if (grow < M && gcol < N) *reinterpret_cast<uint4*>(X + grow * ldx + zcol) = o;
          }
        }
      }
      wave_lds_sync();
    }
  }
}

// everything a launch needs (the epilogues take what they need of it)
struct Args {
  const bf16_t *A, *B;
  void* C;
  const bf16_t* R;
  int M, N, K;
  int64_t lda, ldb, ldc, ldr;
  uint32_t ab, bb;
  hipStream_t st;
  int col0;
  void* X;
  int64_t ldx;
  int xf;
  SegArgs segs;
  RopeArgs rope;
  SplitArgs split;
};

template <int WTM, int WTN, int WGM, bool ATR, bool BTR, int EPI, bool SEG, int NS, bool SPLIT>
hipError_t launch_t16_as(const Args& a) {
  using G = Cfg<WTM, WTN, WGM, ATR, BTR, EPI, SEG, NS>;
  auto kern = gemm_t16_kernel<WTM, WTN, WGM, ATR, BTR, EPI, SEG, NS, SPLIT>;
  static std::atomic<uint64_t> lds_raised{0};
  if (hipError_t e = mls::raise_lds_limit(reinterpret_cast<const void*>(kern), G::LDS, lds_raised)) return e;
  if constexpr (SEG) {
    SegArgs segs = a.segs;
    int tiles = 0;
    for (int i = 0; i < segs.n; i++) {
      SegProblem& p = segs.p[i];
      p.tiles_m = (p.M + G::BM - 1) / G::BM;
      p.tile0 = tiles;
      tiles += p.tiles_m * ((p.N + G::BN - 1) / G::BN);
    }
    hipLaunchKernelGGL(kern, dim3(unsigned(tiles + segs.cs.wgs)), dim3(256), G::LDS, a.st, a.A, a.B, a.C, a.R, a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.ldr,
                       a.ab, a.bb, 0, a.col0, a.X, a.ldx, a.xf, segs, a.rope, SplitArgs{nullptr, nullptr, 1});
  } else {
    const int tm = (a.M + G::BM - 1) / G::BM, tn = (a.N + G::BN - 1) / G::BN;
    hipLaunchKernelGGL(kern, dim3(unsigned(tm) * tn * (SPLIT ? a.split.parts : 1)), dim3(256), G::LDS, a.st, a.A, a.B, a.C, a.R, a.M, a.N, a.K, a.lda, a.ldb, a.ldc,
                       a.ldr, a.ab, a.bb, tm, a.col0, a.X, a.ldx, a.xf, NoSegs{}, a.rope, a.split);
  }
  return hipGetLastError();
}

template <int WTM, int WTN, int WGM, bool ATR, bool BTR, int EPI, bool SEG, int NS>
hipError_t launch_t16(const Args& a) {
  if (a.split.parts <= 1) return launch_t16_as<WTM, WTN, WGM, ATR, BTR, EPI, SEG, NS, false>(a);
  if constexpr (!ATR && !BTR && (EPI != E_DSWIGLU || WTM * WTN < 16)) {
    if (a.split.parts > (WTM * WTN >= 32 ? 2 : 8) || a.split.parts > (a.K + BK - 1) / BK || !a.split.sums) return hipErrorInvalidValue;
    return launch_t16_as<WTM, WTN, WGM, ATR, BTR, EPI, SEG, NS, true>(a);
  }
  return hipErrorInvalidValue;
}

// the tile sizes of one form; the fused epilogues need 64 (gate/up) or 128 (head) columns per wavefront
template <bool ATR, bool BTR, int EPI, bool SEG>
hipError_t run(int tile, const Args& a) {
  if constexpr (EPI == E_ROPE) {
    if (tile == mls::T16_256x128) return launch_t16<4, 8, 4, ATR, BTR, EPI, SEG, 3>(a);
    if (tile == mls::T16_128x128) return launch_t16<2, 8, 4, ATR, BTR, EPI, SEG, 4>(a);
    return launch_t16<1, 8, 4, ATR, BTR, EPI, SEG, 3>(a);
  } else {
    if (tile == mls::T16_256x128) return launch_t16<8, 4, 2, ATR, BTR, EPI, SEG, 3>(a);
    if (tile == mls::T16_128x128) return launch_t16<4, 4, 2, ATR, BTR, EPI, SEG, 4>(a);
    if constexpr (EPI == E_SWIGLU) {
      return launch_t16<2, 4, 2, ATR, BTR, EPI, SEG, 3>(a);
    } else {
      if (tile == mls::T16_128x64) return launch_t16<4, 2, 2, ATR, BTR, EPI, SEG, 3>(a);
      return launch_t16<2, 2, 2, ATR, BTR, EPI, SEG, 3>(a);
    }
  }
}

}  // namespace

namespace mls {

hipError_t gemm_t16(const T16Problem& p, int tile, hipStream_t st) {
  if (p.M <= 0 || p.N <= 0 || p.K <= 0 || p.nseg < 0 || p.nseg > MAX_SEGS) return hipErrorInvalidValue;
  Args a = {};
  a.A = (const bf16_t*)p.A; a.B = (const bf16_t*)p.B; a.C = p.C; a.R = (const bf16_t*)p.R;
  a.M = p.M; a.N = p.N; a.K = p.K;
  a.lda = p.lda; a.ldb = p.ldb; a.ldc = p.ldc; a.ldr = p.ldr;
  a.ab = p.ab; a.bb = p.bb;
  a.st = st;
  a.col0 = p.col0;
  a.X = p.X; a.ldx = p.ldx; a.xf = p.xf;
  a.rope = {p.cos_tab, p.sin_tab, p.seq, p.rot_cols, p.head_dim};
  a.split = {p.split.sums, p.split.state, p.parts > 1 ? p.parts : 1};
  switch (p.form) {
    case T16_NN: return run<false, true, E_BF16, false>(tile, a);
    case T16_NT: return run<false, false, E_BF16, false>(tile, a);
    case T16_TN: return run<true, true, E_F32, false>(tile, a);
    case T16_TN_SEGS: return gemm_t16_group(&p, 1, tile, st);
    case T16_NT_SWIGLU: return run<false, false, E_SWIGLU, false>(tile, a);
    case T16_NT_ROPE: return run<false, false, E_ROPE, false>(tile, a);
    case T16_NT_DSWIGLU: return run<false, false, E_DSWIGLU, false>(tile, a);
  }
  return hipErrorInvalidValue;
}

hipError_t gemm_t16_group(const T16Problem* p, int n, int tile, hipStream_t st, const Colsum& cs) {
  if (n < 1 || n > MAX_T16_GROUP) return hipErrorInvalidValue;
  Args a = {};
  a.K = p[0].K;
  a.ldx = p[0].ldx;
  a.st = st;
  a.segs.nseg = p[0].nseg;
  a.segs.n = n;
  a.segs.cs = cs;
  for (int i = 0; i < n; i++) {
    const T16Problem& q = p[i];
    if (q.form != T16_TN_SEGS || q.K != a.K || q.nseg != a.segs.nseg || q.ldx != a.ldx || q.M <= 0 || q.N <= 0 || q.K <= 0 || q.nseg < 1 ||
        q.nseg > MAX_SEGS)
      return hipErrorInvalidValue;
    SegProblem& g = a.segs.p[i];
    for (int j = 0; j < q.nseg; j++) {
      g.a[j] = (const bf16_t*)q.seg_a[j];
      g.b[j] = (const bf16_t*)q.seg_b[j];
    }
    g.C = q.C;
    g.lda = q.lda; g.ldb = q.ldb; g.ldc = q.ldc;
    g.a_bytes = q.ab; g.b_bytes = q.bb;
    g.M = q.M; g.N = q.N; g.col0 = q.col0; g.xf = q.xf;
  }
  return run<true, true, E_F32, true>(tile, a);
}

}  // namespace mls
