// Which kernels run a bf16 contraction: whole rounds of 256x256 tiles on gemm_bf16_m16.hip, the rest on the smaller tiles
// of gemm_bf16_t16.hip.  Host code only.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int CUS = 256;

struct Plan {
  int n1;         // leading columns (a multiple of 256, possibly 0, or all) that run on 256x256 tiles
  int n1_parts;   // workgroups per tile there, each over a share of the contraction (1 or 2)
  int tile;       // T16_*: how the columns from n1 on run
  int parts;      // workgroups per tile there
  double us;
};

// Estimated microseconds of M x N outputs over a contraction of `it` 64-deep k-tiles.
//   256x256, 256x128, 128x128: one workgroup per CU.  A round costs base + it * c; c depends on how full the chip is (clock and
//     L2 bandwidth are shared).
//   128x64, 64x64: two and three workgroups per CU.  A lone workgroup is a chain of waits; past that the loads of a CU's
//     workgroups add up.  deep: what a long contraction costs where many of them share a CU, whose panels leave the L2 between
//     one k-tile and the next.  top: how far the fullest CU counts beyond the average one, since the last of its workgroups ends
//     the launch (128x64, us per k-tile: 0.29 with 254 tiles, 0.45 with 258, 0.56 with 490, 0.79 with 513).  By the average alone
//     1141 x 2152 over 5248 (306 tiles of 128x64, 48 us) did not get its 128x128 tiles (36 us), nor 1650 x 1280 over 11840 its
//     own (96 instead of 73, 66 shared out).
// Results in bf16 (NN, NT): fitted to stand-alone timings of every tile size, whole and shared out, at 426 shapes (64 to 8192
// tokens, widths 192 to 8192, contractions of 192 to 50304, N(0,1) operands), top to these and 320 more.  The plan with the
// smallest estimate is on average 0.8 % slower than the fastest one measured at all of them, 0.2 % among the whole ones; the worst
// is 19 % (448 x 4392 over 25472, whole: 189 us instead of 159).
// Results in fp32 (TN): twice the bytes where they are stored, four times where they are added to, which a tile that has its CU
// for itself moves while the matrix cores idle: fitted apart, to the weight gradients of 130 layers inside a stage (48 to 5400
// tokens, hidden 192 to 8192), every tile size, in one launch and apart, when results still left the kernels as pieces of rows.
// Leaving as whole rows they cost less (f32_results in common.h; a round of added 256x256 results about 29 us instead of the 47.9
// below), and the choice is on average this far above the fastest measured now: 0.9 % for a product by itself (313 shapes, stored and
// added); between a shared launch and launches apart 3.7 % where results are added to and 2.3 % where they are stored (80 layers of
// these ranges; the worst 20 %, hidden 4744 over 541 tokens 747 us instead of 621, and 25 %, hidden 3624 over 167 tokens 125 instead of 100).
// The fused epilogues have one 64x128 kernel where the plan says 128x64 or 64x64.
enum { TILE_M16 = -1 };
enum Result { R_BF16, R_F32_STORE, R_F32_ADD };
constexpr double LAUNCH_GAP = 1.5;
int64_t tiles_of(int tile, int64_t M, int64_t N) {
  const int bm = tile == mls::T16_64x64 ? 64 : tile == TILE_M16 || tile == mls::T16_256x128 ? 256 : 128;
  const int bn = tile == TILE_M16 ? 256 : tile == mls::T16_256x128 || tile == mls::T16_128x128 ? 128 : 64;
  return ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
}
double estimate(Result res, int tile, int64_t w, int64_t it) {  // w tiles
  if (tile == TILE_M16 || tile == mls::T16_256x128 || tile == mls::T16_128x128) {
    // share: the part of `base` that a nearly empty round pays
    struct Round { double lo, hi, base, share; };
    const Round rounds[3][3] = {{{0.92, 1.38, 8.5, 1}, {0.56, 0.80, 5.7, 1}, {0.33, 0.45, 4.7, 1}},
                                {{0.945, 1.269, 17.1, 0.9}, {0.719, 0.829, 10.0, 1}, {0.464, 0.529, 6.2, 1}},
                                {{1.021, 1.236, 47.9, 0.5}, {0.741, 0.823, 23.1, 0.63}, {0.454, 0.534, 12.1, 0.74}}};
    const Round& r = rounds[res][tile == TILE_M16 ? 0 : tile == mls::T16_256x128 ? 1 : 2];
    const double part = double(w % CUS) / CUS, full = double(w / CUS) * (double(it) * r.hi + r.base);
    return part > 0 ? full + double(it) * (r.lo + (r.hi - r.lo) * part) + r.base * (r.share + (1 - r.share) * part) : full;
  }
  struct Load { double lone, c0, c1, base, each, deep, top; };  // each: per workgroup of a CU; deep, top: see above
  const Load loads[3][2] = {{{0.265, 0.047, 0.291, 4.1, 0, 0.053, 0.22}, {0.212, 0.105, 0.150, 3.1, 0, 0.153, 0.33}},
                            {{0.344, 0.078, 0.319, 4.4, 2.11}, {0.266, 0.121, 0.195, 3.5, 1.05}},
                            {{0.366, 0.063, 0.316, 5.0, 4.24}, {0.286, 0.076, 0.200, 3.7, 1.97}}};
  const Load& l = loads[res][tile == mls::T16_128x64 ? 0 : 1];
  const double load = double(w) / CUS, felt = load + l.top * (double((w + CUS - 1) / CUS) - load);
  double deep = 1;
  if (load > 2 && it > 64) deep += l.deep * std::min(1.0, load / 2 - 1) * std::min(std::log2(double(it) / 64), 2.5);
  const double loop = double(it) * std::max(l.lone, (l.c0 + l.c1 * felt) * deep);
  return loop + (res == R_BF16 ? l.base * std::max(1.0, load / 2) : l.base + l.each * load);
}
double estimate(Result res, int tile, int64_t M, int64_t N, int64_t it) { return estimate(res, tile, tiles_of(tile, M, N), it); }

// Sharing a tile's contraction out over `parts` workgroups (NT products of a caller with a workspace): the time of that many
// tiles over a share of it each, and of the exchange, which grows with the parts to add and with what all of them move.
// At 426 shapes (64 to 8192 tokens, widths 192 to 8192, contractions of 192 to 50304) the plan takes 134 of them apart, which
// then run 1.42 times as fast on average; the worst choice among these loses 6 % (187 x 232 x 1536: 8.5 us, whole 8.0).  us: 100 x 1024 x 50304 172 -> 34 (64x64 in 8),
// 700 x 1536 x 8192 40 -> 31 (128x128 in 3), 2048 x 4096 x 22016 310 -> 254 (256x256 in 2), 2048 x 4096 x 4096 stays 59 (75).
constexpr int MAX_PARTS = 8;
double join_us(int tile, int parts, int64_t w) {
  struct Join { double base, part, load; };
  const Join joins[5] = {{4.2, 2.1, 3.7}, {2.4, 1.2, 4.0}, {1.6, 0.96, 3.0}, {1.37, 0.78, 2.36}, {1.2, 0.66, 1.25}};
  const Join& j = joins[tile + 1];
  return j.base + j.part * parts + j.load * double(w) / CUS;
}
// the sums they leave, 0 if a workspace does not hold them (a shape's own tile sizes: the fused forms have a 64x128 kernel for
// both of the smallest)
int64_t split_floats(int form, int tile, int parts, int64_t M, int64_t N, int64_t it) {
  if (parts > (tile == TILE_M16 || tile == mls::T16_256x128 ? 2 : MAX_PARTS) || it < 4 * parts) return 0;
  int bm = 256, bn = 256;
  if (tile != TILE_M16) mls::t16_tile_size(form, tile, bm, bn);
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn), floats = tiles * (parts == 2 ? 1 : parts) * bm * bn;
  return tiles <= mls::SPLIT_TILES && floats <= mls::SPLIT_FLOATS ? floats : 0;
}

// m16: the 256x256 kernel takes the problem (the fused forms need whole 64-deep k-tiles there); split: tiles may be shared out
Plan plan(Result res, int form, int M, int N, int64_t K, bool m16, bool split) {
  const int64_t it = (K + 63) / 64, tm = (M + 255) / 256, tn = (N + 255) / 256;
  const int n1 = int(tm * tn / CUS * CUS / tm) * 256;  // columns that whole rounds of 256x256 tiles cover
  Plan best = {N, 1, mls::T16_256x128, 1, 0};
  double t = m16 ? estimate(res, TILE_M16, M, N, it) : HUGE_VAL;
  auto shared = [&](int tile, int parts, int64_t n) {
    const int64_t w = tiles_of(tile, M, n) * parts;
    return estimate(res, tile, w, (it + parts - 1) / parts) + join_us(tile, parts, w);
  };
  const int most = !split ? 1 : int(std::max<int64_t>(1, std::min<int64_t>(MAX_PARTS, it / 4)));  // four k-tiles or more each
  for (int tile : {mls::T16_256x128, mls::T16_128x128, mls::T16_128x64, mls::T16_64x64})
    for (int parts = 1; parts <= most; parts++) {
      if (parts == 1 || split_floats(form, tile, parts, M, N, it)) {
        const double all = parts == 1 ? estimate(res, tile, M, N, it) : shared(tile, parts, N);
        if (all < t) {
          t = all;
          best = {0, 1, tile, parts, 0};
        }
      }
      if (!m16 || n1 == 0 || n1 >= N || (parts > 1 && !split_floats(form, tile, parts, M, N - n1, it))) continue;
      const double rest = parts == 1 ? estimate(res, tile, M, N - n1, it) : shared(tile, parts, N - n1);
      const double both = estimate(res, TILE_M16, M, n1, it) + rest + LAUNCH_GAP;
      if (both < t) {
        t = both;
        best = {n1, 1, tile, parts, 0};
      }
    }
  if (split && m16 && K % 64 == 0 && split_floats(form, TILE_M16, 2, M, N, it)) {
    const double all = shared(TILE_M16, 2, N);
    if (all < t) {
      t = all;
      best = {N, 2, mls::T16_256x128, 1, 0};
    }
  }
  best.us = t;
  return best;
}

// the columns from n1 on of a problem whose B is given for all of them
mls::T16Problem columns_from(mls::T16Problem p, int n1) {
  const bool nt = p.form == mls::T16_NT || p.form == mls::T16_NT_SWIGLU || p.form == mls::T16_NT_ROPE;
  if (nt) {
    p.B = (const uint16_t*)p.B + int64_t(n1) * p.ldb;
    p.bb = uint32_t(int64_t(p.N - n1) * p.ldb * 2);
  } else {
    if (p.B) p.B = (const uint16_t*)p.B + n1;
    for (int i = 0; i < p.nseg; i++) p.seg_b[i] = (const uint16_t*)p.seg_b[i] + n1;
  }
  p.N -= n1;
  p.col0 = n1;
  return p;
}

bool fused(int form) { return form == mls::T16_NT_SWIGLU || form == mls::T16_NT_ROPE; }

Plan plan(int form, bool store, int M, int N, int64_t K, bool split = false) {
  const Result res = form != mls::T16_TN && form != mls::T16_TN_SEGS ? R_BF16 : store ? R_F32_STORE : R_F32_ADD;
  return plan(res, form, M, N, K, !fused(form) || K % 64 == 0, split && (form == mls::T16_NT || fused(form)));
}

// `big(n1, space)` runs the leading n1 columns on 256x256 tiles, shared out where it gets a space
template <class Big>
hipError_t run(const mls::T16Problem& p, hipStream_t st, Big&& big) {
  const int64_t depth = p.nseg > 0 ? (int64_t(p.K) + 63) / 64 * 64 * p.nseg : p.K;  // (every piece ends with a k-tile of its own)
  const Plan pl = plan(p.form, p.form == mls::T16_TN_SEGS && p.ldx != 0, p.M, p.N, depth, p.split.sums != nullptr);
  if (pl.n1 > 0)
    if (hipError_t e = big(pl.n1, pl.n1_parts > 1 ? &p.split : nullptr)) return e;
  if (pl.n1 == p.N) return hipSuccess;
  mls::T16Problem rest = columns_from(p, pl.n1);
  rest.parts = pl.parts;
  return mls::gemm_t16(rest, pl.tile, st);
}

mls::T16Problem problem(int form, const void* A, const void* B, void* C, int M, int N, int K, int64_t lda, int64_t ldb,
                        int64_t ldc, uint32_t ab, uint32_t bb) {
  mls::T16Problem p = {};
  p.form = form;
  p.A = A; p.B = B; p.C = C;
  p.M = M; p.N = N; p.K = K;
  p.lda = lda; p.ldb = ldb; p.ldc = ldc;
  p.ab = ab; p.bb = bb;
  return p;
}

mls::T16Problem tn_problem(const mls::TnProduct& t, int nseg, int kseg, bool overwrite) {
  mls::T16Problem p = problem(mls::T16_TN_SEGS, t.A[0], nullptr, t.C, t.M, t.N, kseg, t.lda, t.ldb, t.ldc, uint32_t(int64_t(kseg) * t.lda * 2),
                              uint32_t(int64_t(kseg) * t.ldb * 2));
  p.nseg = nseg;
  for (int i = 0; i < nseg; i++) {
    p.seg_a[i] = t.A[i];
    p.seg_b[i] = t.B[i];
  }
  p.ldx = overwrite ? 1 : 0;
  p.xf = t.gu_f;
  return p;
}

}  // namespace

namespace mls {

// true if the DMA kernels can run this problem: every operand (plus one tile of slack) addressable with a 31-bit byte
// offset
bool gemm_bf16_dma_ok(int mode, int M, int N, int K, int64_t lda, int64_t ldb) {
  const int64_t a_rows = mode == GEMM_TN ? K : M, b_rows = mode == GEMM_NT ? N : K;
  const int64_t lim = int64_t(1) << 31;
  return (a_rows + 512) * lda * 2 < lim && (b_rows + 512) * ldb * 2 < lim && K > 0;
}

hipError_t gemm_bf16_dma(int mode, const void* A, const void* B, void* C, const void* R, int M, int N, int K,
                         int64_t lda, int64_t ldb, int64_t ldc, int64_t ldr, hipStream_t st, const SplitSpace& split) {
  if (M == 0 || N == 0) return hipSuccess;
  const int64_t a_rows = mode == GEMM_TN ? K : M, b_rows = mode == GEMM_NT ? N : K;
  const uint32_t ab = uint32_t(a_rows * lda * 2), bb = uint32_t(b_rows * ldb * 2);
  T16Problem p = problem(mode == GEMM_NN ? T16_NN : mode == GEMM_NT ? T16_NT : T16_TN, A, B, C, M, N, K, lda, ldb, ldc, ab, bb);
  p.R = R;
  p.ldr = ldr;
  p.split = split;
  return run(p, st, [&](int n1, const SplitSpace* sp) { return gemm_m16(mode, A, B, C, R, M, n1, K, lda, ldb, ldc, ldr, ab, bb, st, sp); });
}

void t16_tile_size(int form, int tile, int& rows, int& cols) {
  rows = tile == T16_256x128 ? 256 : tile == T16_64x64 || (fused(form) && tile == T16_128x64) ? 64 : 128;
  cols = tile == T16_256x128 || tile == T16_128x128 || fused(form) ? 128 : 64;
}

GemmPlan gemm_bf16_plan(int form, int M, int N, int K, bool split) {
  const Plan p = plan(form, false, M, N, K, split);
  GemmPlan g = {p.n1, 0, 0, p.n1_parts, p.parts};
  if (p.n1 < N) t16_tile_size(form, p.tile, g.tile_rows, g.tile_cols);
  return g;
}

int64_t gemm_split_floats(int form, int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0) return 0;
  const Plan p = plan(form, false, M, N, K, true);
  const int64_t it = (int64_t(K) + 63) / 64;
  if (p.n1_parts > 1) return split_floats(form, TILE_M16, p.n1_parts, M, N, it);
  return p.parts > 1 ? split_floats(form, p.tile, p.parts, M, N - p.n1, it) : 0;
}

bool gemm_tn_segments_ok(int kseg, int64_t lda, int64_t ldb) { return gemm_bf16_dma_ok(GEMM_TN, 8, 8, kseg, lda, ldb); }

// C[M,N] += sum_i A_i[kseg,M]^T * B_i[kseg,N] (fp32 C), the contraction of all pieces accumulated in registers and
// added to C once: the weight gradient of several micro-batches in one launch.  nseg <= 16.
hipError_t gemm_bf16_tn_segments(const void* const* A, const void* const* B, int nseg, void* C, int M, int N, int kseg,
                                 int64_t lda, int64_t ldb, int64_t ldc, hipStream_t st, int gu_f, bool overwrite) {
  if (M == 0 || N == 0 || nseg == 0 || kseg == 0) return hipSuccess;
  if (nseg > 16 || (gu_f > 0 && (gu_f % 8 || N != 2 * gu_width(gu_f)))) return hipErrorInvalidValue;
  const T16Problem p = tn_problem({A, B, C, M, N, lda, ldb, ldc, gu_f}, nseg, kseg, overwrite);
  return run(p, st, [&](int n1, const SplitSpace*) { return gemm_m16_group(&p, &n1, 1, st); });
}

// One launch of one tile size for all of them, or a launch (or two) for each, by the same estimates.  Small layers win the
// empty last rounds and the launches, large ones keep their whole rounds of 256x256 tiles.  The four weight gradients of a
// layer, apart -> in one (us): hidden 256, 256 tokens 25 -> 9; 1024 / ffn 2728, 2000 tokens 112 -> 80; 768, 2 x 1024 tokens
// 80 -> 45; 1536, 700 tokens 125 -> 97 (the fastest tile: 89); 512, 4 x 4096 tokens 387 -> 157; 3072, 600 tokens 422 -> 420.
// 256x256 tiles: together their partly empty last rounds become one, and where that one would be nearly empty a product's last columns
// that make it up go to smaller tiles (2048 / 5504, 2 x 2048 tokens: 776 tiles as 768 and 2048 x 256 columns on 64x64 ones; a step of that layer
// 1 652 -> 1 602 us, hidden 5120 / 13824 over 2 x 4096 0.7 % faster; over 4 x 4096 tokens at 4096 / 11008, at the power limit, equal; 25 layers
// of hidden 2048 to 5888 the weight gradients 0.87 and a step 0.97 of the time apart, none slower).  From two rounds of them and 32 k-tiles on, where
// that was first measured.  It is not where they stop paying: of 187 layers below either line (hidden 512 to 6200) the estimates would take them
// together with 0.85 of the time for the weight gradients and 0.97 for a step, 11 of them slower by up to 2.8 % (contractions of less than 16 k-tiles,
// 257 to 320 tiles).
TnGroupPlan gemm_bf16_tn_group_plan(const TnProduct* p, int n, int nseg, int kseg, bool overwrite) {
  const int64_t it = int64_t(nseg) * ((kseg + 63) / 64), depth = it * 64;
  const Result res = overwrite ? R_F32_STORE : R_F32_ADD;
  double least = -LAUNCH_GAP;
  int64_t big = 0;
  for (int i = 0; i < n; i++) {
    if (p[i].M <= 0 || p[i].N <= 0) continue;
    least += LAUNCH_GAP + plan(T16_TN_SEGS, overwrite, p[i].M, p[i].N, depth).us;
    big += tiles_of(TILE_M16, p[i].M, p[i].N);
  }
  TnGroupPlan best = {false, -1, -1, 0, 0};
  auto consider = [&](double t, const TnGroupPlan& g) {
    if (t < least) least = t, best = g;
  };
  for (int tile : {T16_256x128, T16_128x128, T16_128x64, T16_64x64}) {
    int64_t w = 0;
    for (int i = 0; i < n; i++) w += tiles_of(tile, p[i].M, p[i].N);
    consider(estimate(res, tile, w, it), {true, tile, -1, 0, 0});
  }
  if (big < 2 * CUS || it < 32) return best;
  consider(estimate(res, TILE_M16, big, it), {true, -1, -1, 0, 0});
  for (int i = 0; i < n; i++) {
    if (p[i].M <= 0 || p[i].N <= 0) continue;
    const int64_t tm = (p[i].M + 255) / 256, tn = (p[i].N + 255) / 256, drop = (big % CUS + tm - 1) / tm;  // tile columns that end the last round
    if (drop < 1 || drop >= tn || big - drop * tm < CUS) continue;
    const int n1 = int(tn - drop) * 256;
    for (int rest : {T16_256x128, T16_128x128, T16_128x64, T16_64x64})
      consider(estimate(res, TILE_M16, big - drop * tm, it) + LAUNCH_GAP + estimate(res, rest, p[i].M, p[i].N - n1, it), {true, -1, i, n1, rest});
  }
  return best;
}

hipError_t gemm_bf16_tn_group(const TnProduct* p, int n, const TnGroupPlan& plan, int nseg, int kseg, hipStream_t st, bool overwrite, const Colsum& cs) {
  if (nseg == 0 || kseg == 0) return hipSuccess;
  if (n < 1 || n > MAX_T16_GROUP || nseg > 16 || !plan.together) return hipErrorInvalidValue;
  T16Problem q[MAX_T16_GROUP];
  int n1[MAX_T16_GROUP], m = 0, split = -1;
  for (int i = 0; i < n; i++) {
    if (p[i].gu_f > 0 && (p[i].gu_f % 8 || p[i].N != 2 * gu_width(p[i].gu_f))) return hipErrorInvalidValue;
    if (p[i].M == 0 || p[i].N == 0) continue;
    if (i == plan.split) split = m;
    n1[m] = i == plan.split ? plan.n1 : p[i].N;
    q[m++] = tn_problem(p[i], nseg, kseg, overwrite);
  }
  if (m == 0) return hipSuccess;
  if (plan.tile >= 0) return gemm_t16_group(q, m, plan.tile, st, cs);
  if (hipError_t e = gemm_m16_group(q, n1, m, st, cs)) return e;
  if (split < 0) return hipSuccess;
  const T16Problem rest = columns_from(q[split], plan.n1);
  return gemm_t16_group(&rest, 1, plan.rest, st);
}

bool gemm_swiglu_ok(int M, int f, int K, int64_t lda, int64_t ldw) {
  return f > 0 && f % 32 == 0 && gemm_bf16_dma_ok(GEMM_NT, M, 2 * f, K, lda, ldw);
}

hipError_t gemm_bf16_swiglu(const void* A, const void* W, void* GU, void* Z, int M, int f, int K, int64_t lda,
                            int64_t ldw, int64_t ldgu, int64_t ldz, hipStream_t st, const SplitSpace& split) {
  if (M == 0 || f == 0) return hipSuccess;
  if (!gemm_swiglu_ok(M, f, K, lda, ldw)) return hipErrorInvalidValue;
  const uint32_t ab = uint32_t(int64_t(M) * lda * 2), wb = uint32_t(int64_t(2 * f) * ldw * 2);
  T16Problem p = problem(T16_NT_SWIGLU, A, W, GU, M, 2 * f, K, lda, ldw, ldgu, ab, wb);
  p.X = Z;
  p.ldx = ldz;
  p.split = split;
  return run(p, st, [&](int n1, const SplitSpace* sp) { return gemm_m16_swiglu(A, W, GU, Z, M, n1, K, lda, ldw, ldgu, ldz, ab, wb, st, sp); });
}

// Not on 256x256 tiles, whose only wavefront per SIMD would move the three times as many bytes with the matrix cores idle; on the smaller ones
// it saves a pass over dZ and a launch.  Microseconds saved of a layer's step of 100 to 800, mean of 28 shapes for each tile: 64x64 1.9, 128x64 2.1,
// 128x128 1.9, 256x128 3.0, shared out over the contraction 64x64 0.8 and 128x64 0.9, but 128x128 -0.3 (in three -1.3): there the one workgroup
// that adds up a tile runs its epilogue after the others have left.
bool gemm_dswiglu_ok(int M, int f, int K, int64_t lda, int64_t ldw, bool split) {
  if (f <= 0 || f % 8 || !gemm_bf16_dma_ok(GEMM_NT, M, f, K, lda, ldw)) return false;
  const Plan pl = plan(T16_NT, false, M, f, K, split);
  return pl.n1 == 0 && (pl.parts == 1 || pl.tile == T16_128x64 || pl.tile == T16_64x64);
}

hipError_t gemm_bf16_dswiglu(const void* dY, const void* W, const void* GU, void* DGU, int M, int f, int K, int64_t lda, int64_t ldw,
                             int64_t ldgu, int64_t lddgu, hipStream_t st, const SplitSpace& split) {
  if (M == 0 || f == 0) return hipSuccess;
  if (!gemm_dswiglu_ok(M, f, K, lda, ldw, split.sums != nullptr)) return hipErrorInvalidValue;
  const Plan pl = plan(T16_NT, false, M, f, K, split.sums != nullptr);
  T16Problem p = problem(T16_NT_DSWIGLU, dY, W, DGU, M, f, K, lda, ldw, lddgu, uint32_t(int64_t(M) * lda * 2), uint32_t(int64_t(f) * ldw * 2));
  p.R = GU;
  p.ldr = ldgu;
  p.split = split;
  p.parts = pl.parts;
  return gemm_t16(p, pl.tile, st);
}

bool gemm_rope_ok(int M, int N, int K, int64_t lda, int64_t ldw, int seq, int rot_cols, int head_dim) {
  return (head_dim == 64 || head_dim == 128) && seq > 0 && rot_cols >= 0 && rot_cols <= N && rot_cols % head_dim == 0 &&
         N % head_dim == 0 && gemm_bf16_dma_ok(GEMM_NT, M, N, K, lda, ldw);
}

hipError_t gemm_bf16_rope(const void* A, const void* W, void* C, int M, int N, int K, int64_t lda, int64_t ldw, int64_t ldc,
                          const float* cos_tab, const float* sin_tab, int seq, int rot_cols, int head_dim, hipStream_t st,
                          const SplitSpace& split) {
  if (M == 0 || N == 0) return hipSuccess;
  if (!cos_tab || !sin_tab || !gemm_rope_ok(M, N, K, lda, ldw, seq, rot_cols, head_dim)) return hipErrorInvalidValue;
  const uint32_t ab = uint32_t(int64_t(M) * lda * 2), wb = uint32_t(int64_t(N) * ldw * 2);
  T16Problem p = problem(T16_NT_ROPE, A, W, C, M, N, K, lda, ldw, ldc, ab, wb);
  p.cos_tab = cos_tab;
  p.sin_tab = sin_tab;
  p.seq = seq;
  p.rot_cols = rot_cols;
  p.head_dim = head_dim;
  p.split = split;
  return run(p, st, [&](int n1, const SplitSpace* sp) {
    return gemm_m16_rope(A, W, C, M, n1, K, lda, ldw, ldc, ab, wb, cos_tab, sin_tab, seq, rot_cols, head_dim, st, sp);
  });
}

}  // namespace mls
