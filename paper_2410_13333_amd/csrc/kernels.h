// Host-side launchers of the HIP kernels of the decoder-stage library.  Every launcher enqueues on `st`,
// never synchronises and returns the launch status.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace mls {

enum { GEMM_NN = 0, GEMM_NT = 1, GEMM_TN = 2 };
enum { DT_BF16 = 0, DT_FP32 = 1 };

// records `msg` as the calling thread's mls_last_error text and returns `code` (stage.hip)
int set_error(int code, const char* msg);

// Raises a kernel's dynamic-LDS limit, once per device (the attribute belongs to the function on the current
// device).  `done` is the launcher's own bit mask of devices already served; racing threads at worst set it twice.
inline hipError_t raise_lds_limit(const void* kern, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = uint64_t(1) << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// Column sums: out[c] (+)= sum over nblocks rows of partial[.][h], one or two of them; wgs: workgroups of 256 threads (colsum_block in
// common.h)
struct Colsum {
  const float* partial0;
  float* out0;
  const float* partial1;
  float* out1;
  int nblocks, h, overwrite, wgs;
};

// Workspace of contractions that are shared out over several workgroups per tile (join_parts in common.h); it belongs to the
// launches of one stream.  state: SPLIT_TILES pairs of counters, zero between launches; sums: what the products need
// (gemm_split_floats), at most SPLIT_FLOATS.  Null: none is shared out.
constexpr int64_t SPLIT_FLOATS = int64_t(8) << 20, SPLIT_TILES = 1024;
struct SplitSpace {
  float* sums = nullptr;
  uint32_t* state = nullptr;
};
// one allocation for both: the counters, then the sums; 0 bytes where no product needs it
inline size_t split_bytes(int64_t floats) { return floats > 0 ? size_t(SPLIT_TILES) * 8 + size_t(floats) * 4 : 0; }
inline SplitSpace split_space(void* p) {
  if (!p) return {};
  return {reinterpret_cast<float*>(static_cast<char*>(p) + SPLIT_TILES * 8), static_cast<uint32_t*>(p)};
}

// ---- contractions (gemm_bf16.hip, gemm_f32.hip); modes as documented at mls_gemm; leading dims in elements
// (ldr: row stride of the residual R, ignored when R is null)
hipError_t gemm_bf16(int mode, const void* A, const void* B, void* C, const void* R, int M, int N, int K, int64_t lda,
                     int64_t ldb, int64_t ldc, int64_t ldr, hipStream_t st, const SplitSpace& split = {});
// the two implementations behind gemm_bf16: LDS-DMA main path and the register-staged fallback for operands
// too large for 31-bit buffer offsets
bool gemm_bf16_dma_ok(int mode, int M, int N, int K, int64_t lda, int64_t ldb);
hipError_t gemm_bf16_dma(int mode, const void* A, const void* B, void* C, const void* R, int M, int N, int K,
                         int64_t lda, int64_t ldb, int64_t ldc, int64_t ldr, hipStream_t st, const SplitSpace& split = {});
// What such a problem runs on (form: T16_NN .. T16_NT_ROPE below): the leading columns that get 256x256 tiles, the size of
// the tiles behind them (0 x 0 if there are none), and, of a caller with a SplitSpace, the workgroups per tile of either.
// Host only.
struct GemmPlan { int big_cols, tile_rows, tile_cols, big_parts, parts; };
GemmPlan gemm_bf16_plan(int form, int M, int N, int K, bool split = false);
int64_t gemm_split_floats(int form, int M, int N, int K);  // what it needs of a SplitSpace (0: nothing).  Host only.
void t16_tile_size(int form, int tile, int& rows, int& cols);  // T16_* of a form in rows and columns
// weight gradient of several micro-batches in one launch: C[M,N] += sum_i A_i[kseg,M]^T * B_i[kseg,N], C fp32,
// at most 16 pieces, all with the same strides; true if the operands fit the DMA path's 31-bit offsets
bool gemm_tn_segments_ok(int kseg, int64_t lda, int64_t ldb);
// gu_f > 0: the N = 2 gu_width(gu_f) columns of the B pieces are in the interleaved gate/up order and C is in the public one
// overwrite: C = instead of C += (the fp32 gradient is then not read)
hipError_t gemm_bf16_tn_segments(const void* const* A, const void* const* B, int nseg, void* C, int M, int N, int kseg,
                                 int64_t lda, int64_t ldb, int64_t ldc, hipStream_t st, int gu_f = 0,
                                 bool overwrite = false);
// several such products (n <= MAX_T16_GROUP) over pieces of the same depth
struct TnProduct {
  const void *const *A, *const *B;
  void* C;
  int M, N;
  int64_t lda, ldb, ldc;
  int gu_f;
};
// How they run where one launch for all of them fills the chip better than a launch (or two) for each (together).  tile >= 0: all on tiles of
// that size (T16_*); else 256x256 tiles but for the columns from n1 on of product `split` (if >= 0), which get tiles of size `rest` in a
// launch of their own.  Host only.
struct TnGroupPlan {
  bool together;
  int tile, split, n1, rest;
};
TnGroupPlan gemm_bf16_tn_group_plan(const TnProduct* p, int n, int nseg, int kseg, bool overwrite);
// cs: column sums that go along in the same launch (not done if there is nothing to launch: no product, no piece)
hipError_t gemm_bf16_tn_group(const TnProduct* p, int n, const TnGroupPlan& plan, int nseg, int kseg, hipStream_t st, bool overwrite, const Colsum& cs = {});
// the 256x256 tiles of a problem on the 16x16x32 form of the matrix instruction (gemm_bf16_m16.hip); K % 8 == 0 where an
// operand is stored [row][k], % 64 in the two fused forms
hipError_t gemm_m16(int mode, const void* A, const void* B, void* C, const void* R, int M, int N, int K, int64_t lda,
                    int64_t ldb, int64_t ldc, int64_t ldr, uint32_t ab, uint32_t bb, hipStream_t st, const SplitSpace* split = nullptr);
hipError_t gemm_m16_swiglu(const void* A, const void* W, void* GU, void* Z, int M, int N, int K, int64_t lda, int64_t ldw,
                           int64_t ldgu, int64_t ldz, uint32_t ab, uint32_t bb, hipStream_t st, const SplitSpace* split = nullptr);
hipError_t gemm_m16_rope(const void* A, const void* W, void* C, int M, int N, int K, int64_t lda, int64_t ldw, int64_t ldc,
                         uint32_t ab, uint32_t bb, const float* cos_tab, const float* sin_tab, int seq, int rot_cols,
                         int head_dim, hipStream_t st, const SplitSpace* split = nullptr);
// everything else on smaller tiles of the same instruction (gemm_bf16_t16.hip): any K (a multiple of 8 where an operand is
// stored [row][k]).  The columns of B (for NN / TN from pointer B on, for NT from row 0 of B on) are columns col0 .. of C
// (and R, X), which are not offset.
enum { T16_256x128 = 0, T16_128x128 = 1, T16_128x64 = 2, T16_64x64 = 3 };  // (the last two: 64x128 for the fused epilogues)
enum { T16_NN, T16_NT, T16_TN, T16_TN_SEGS, T16_NT_SWIGLU, T16_NT_ROPE, T16_NT_DSWIGLU };
struct T16Problem {
  int form;
  const void *A, *B;
  void* C;
  const void* R;
  int M, N, K;  // T16_TN_SEGS: K = depth of one piece
  int64_t lda, ldb, ldc, ldr;
  uint32_t ab, bb;  // byte lengths of A and B (of one piece)
  int col0;
  void* X;      // SwiGLU: the product; TN forms: ldx != 0 stores instead of adding
  int64_t ldx;
  int xf;       // TN_SEGS: the gate/up width if the columns are in the interleaved order
  int nseg;
  const void *seg_a[16], *seg_b[16];
  const float *cos_tab, *sin_tab;
  int seq, rot_cols, head_dim;
  SplitSpace split;
  int parts;    // > 1: workgroups per tile, each over a share of K (the three NT forms); the space has to hold them
};
hipError_t gemm_t16(const T16Problem& p, int tile, hipStream_t st);
// up to four T16_TN_SEGS problems over pieces of the same number and depth in one launch
constexpr int MAX_T16_GROUP = 4;
hipError_t gemm_t16_group(const T16Problem* p, int n, int tile, hipStream_t st, const Colsum& cs = {});
// the leading n1[i] columns (a multiple of 256, possibly 0, or all) of such problems on 256x256 tiles in one launch
hipError_t gemm_m16_group(const T16Problem* p, const int* n1, int n, hipStream_t st, const Colsum& cs = {});
hipError_t fill_zero_f32(float* p, size_t n, hipStream_t st);
// SwiGLU fused into the gate/up contraction (bf16, f % 32 == 0 here, DMA path).  Interleaved gate/up column order:
// 32 gate columns, the 32 up columns of the same indices, and so on (gu_interleaved_col in common.h).
//   GU[M, 2f] = A[M,K] W[K, 2f] (W and GU interleaved), Z[M, f] = silu(gate) * up
// W is given transposed, [2f][K] (rows in the interleaved order) with row stride ldw.
bool gemm_swiglu_ok(int M, int f, int K, int64_t lda, int64_t ldw);
hipError_t gemm_bf16_swiglu(const void* A, const void* W, void* GU, void* Z, int M, int f, int K, int64_t lda,
                            int64_t ldw, int64_t ldgu, int64_t ldz, hipStream_t st, const SplitSpace& split = {});
// The SwiGLU backward fused into the data gradient of the down-projection (bf16, f % 8 == 0, DMA path), where all of that product runs on
// the smaller tiles, the larger of them whole (gemm_dswiglu_ok; host only): dZ[M, f] = dY[M,K] W[f,K]^T stays in registers,
//   DGU[M, 2f] = (dZ up silu'(gate), dZ silu(gate)), GU and DGU in the interleaved order.
bool gemm_dswiglu_ok(int M, int f, int K, int64_t lda, int64_t ldw, bool split);
hipError_t gemm_bf16_dswiglu(const void* dY, const void* W, const void* GU, void* DGU, int M, int f, int K, int64_t lda, int64_t ldw,
                             int64_t ldgu, int64_t lddgu, hipStream_t st, const SplitSpace& split = {});
// The rotary embedding fused into the q|k|v projection (bf16, DMA path): C[M, N] = A[M,K] W[K,N] rounded to bf16, then
// every head vector (head_dim = 64 or 128 columns) in the columns below rot_cols rotated by the angle of its row's
// position row % seq, pairs (i, i + head_dim/2); cos_tab, sin_tab: [seq][head_dim/2] fp32.
// W is given transposed, [N][K] with row stride ldw.
bool gemm_rope_ok(int M, int N, int K, int64_t lda, int64_t ldw, int seq, int rot_cols, int head_dim);
hipError_t gemm_bf16_rope(const void* A, const void* W, void* C, int M, int N, int K, int64_t lda, int64_t ldw, int64_t ldc,
                          const float* cos_tab, const float* sin_tab, int seq, int rot_cols, int head_dim, hipStream_t st,
                          const SplitSpace& split = {});
bool gemm_f32_large(int M, int N, int K);  // whether such a product runs on 64x64 tiles, not on 32x32 ones.  Host only.
// overwrite (GEMM_TN): C = instead of +=
hipError_t gemm_f32(int mode, const void* A, const void* B, void* C, const void* R, int M, int N, int K, int64_t lda,
                    int64_t ldb, int64_t ldc, int64_t ldr, hipStream_t st, bool overwrite = false);
// The fp32 products with an elementwise step as their epilogue (operands as gemm_f32 takes them): gate|up [M, 2f] and Z = silu(gate) up, both
// stored; C with the head vectors below column rot_cols rotated by row % seq (head_dim a multiple of 16; tables [seq][head_dim/2]);
// the SwiGLU backward of dZ = dY W^T (W [f, K]) from GU [M, 2f].
hipError_t gemm_f32_swiglu(const void* A, const void* W, void* GU, void* Z, int M, int f, int K, int64_t lda, int64_t ldw, int64_t ldgu,
                           int64_t ldz, hipStream_t st);
hipError_t gemm_f32_rope(const void* A, const void* W, void* C, int M, int N, int K, int64_t lda, int64_t ldw, int64_t ldc, const float* cos_tab,
                         const float* sin_tab, int seq, int rot_cols, int head_dim, hipStream_t st);
hipError_t gemm_f32_dswiglu(const void* dY, const void* W, const void* GU, void* DGU, int M, int f, int K, int64_t lda, int64_t ldw,
                            int64_t ldgu, int64_t lddgu, hipStream_t st);
// p[i].C (+)= sum_j p[i].A[j][kseg, M]^T * p[i].B[j][kseg, N] over nseg <= 16 pieces for up to four products, fp32 throughout, and the
// column sums of cs, in one launch (nothing at all without a piece)
int gemm_f32_tn_group_tile(const TnProduct* p, int n);  // rows and columns of its tiles, 32 or 64.  Host only.
hipError_t gemm_f32_tn_group(const TnProduct* p, int n, int nseg, int kseg, hipStream_t st, bool overwrite, const Colsum& cs = {});

// ---- row-wise and elementwise kernels (elementwise.hip); dt selects the storage type; every matrix argument is
// followed by its row stride in elements (all row strides are multiples of 8)
// a = x * r * gamma, r[t] = rsqrt(mean(x^2) + eps) saved as fp32
// copy, if given, receives x with row stride ldc
hipError_t rmsnorm_fwd(int dt, const void* x, int64_t ldx, const void* gamma, void* a, int64_t lda, float* r, int T,
                       int h, float eps, hipStream_t st, void* copy = nullptr, int64_t ldc = 0);
// n matrices of `rows` rows of `bytes`, next_* apart: dense <-> row-padded.  Pointers, strides and bytes are multiples of 16.
hipError_t copy_rows(const void* src, int64_t ld_src, int64_t next_src, void* dst, int64_t ld_dst, int64_t next_dst, int64_t bytes,
                     int rows, int n, hipStream_t st);
// dx = dres + r*(dn - n*mean(dn*n)), dn = da*gamma, n = x*r;  dgamma += sum_t da*n (two-stage, deterministic).
// partial: workspace of rmsnorm_bwd_blocks(T) * h floats.  dres may be null (no residual branch: dx without it).
// overwrite: dgamma = instead of +=.  A sequence of calls over several micro-batches may share one column
// reduction: acc_partial adds this call's row-block sums to those already in `partial` (same T), and only the
// call with `reduce` adds the columns of `partial` into dgamma (dgamma and overwrite are ignored otherwise).
int rmsnorm_bwd_blocks(int T);
hipError_t rmsnorm_bwd(int dt, const void* da, int64_t ld_da, const void* x, int64_t ldx, const void* gamma,
                       const float* r, const void* dres, int64_t ld_dres, void* dx, int64_t ld_dx, float* dgamma,
                       float* partial, int T, int h, hipStream_t st, bool overwrite = false, bool acc_partial = false,
                       bool reduce = true);
// the column reduction of one or (partial1 given) two such sequences over the same T, of a launch of its own or with
// gemm_bf16_tn_group
Colsum rmsnorm_bwd_sums(const float* partial0, float* dgamma0, const float* partial1, float* dgamma1, int T, int h, bool overwrite);
hipError_t rmsnorm_bwd_reduce(const Colsum& cs, hipStream_t st);
// bf16 storage (fp32: gemm_f32_rope): rotate the pairs (i, i+d/2) of the first n_heads heads of every row of u [T, ld] by angle(t % S, i)
hipError_t rope_inplace(void* u, const float* cos_tab, const float* sin_tab, int T, int S, int n_heads, int d, int64_t ld, hipStream_t st);
// bf16 (fp32 storage: gemm_f32_swiglu, gemm_f32_dswiglu)
hipError_t swiglu_fwd(const void* gu, int64_t ld_gu, void* z, int64_t ld_z, int T, int f, hipStream_t st);
hipError_t swiglu_bwd(const void* dz, int64_t ld_dz, const void* gu, int64_t ld_gu, void* dgu, int64_t ld_dgu,
                      int T, int f, hipStream_t st, bool interleaved = false);  // interleaved: gu, dgu in that order
// weights from the counter-based generator: element (r, c) of a rows x cols tensor stored with row stride ld is
// offset + scale*z(seed, tensor, layer, r*cols + c), rounded once
hipError_t fill_normal(int dt, void* out, int64_t rows, int64_t cols, int64_t ld, uint64_t seed, uint32_t tensor,
                       uint32_t layer, double scale, double offset, hipStream_t st, int gu_f = 0);
// Places bf16 parameter matrices: dst[r][c'] = src[r][c] and the transposed copy dst_t[c'][r] = src[r][c] (either may be
// null), c' = c, or its interleaved place if gu_f > 0.  One launch for all of the list.  Columns are multiples of 8, and
// rows too where dst_t is given; all pointers are 16-byte aligned, all row strides multiples of 8.
constexpr int MAX_SPREAD = 6;
struct Spread {
  const void* src;
  int64_t ld_src;
  void* dst;
  int64_t ld_dst;
  void* dst_t;
  int64_t ld_t;
  int rows, cols, gu_f;
};
hipError_t spread_bf16(const Spread* list, int n, hipStream_t st);
// gu_f > 0 above: a [rows, 2 gu_f] gate/up tensor is written in the interleaved column order.  gu_permute moves a
// bf16 [rows, 2f] matrix between the public and the interleaved column order.
hipError_t gu_permute(const void* src, int64_t ld_src, void* dst, int64_t ld_dst, int64_t rows, int f,
                      bool to_interleaved, hipStream_t st);

// ---- attention (attention_bf16.hip, attention_f32.hip).  qkv: [T, q_dim + 2 kv_dim] rows = q heads | k heads | v heads
// (rotary already applied); o: [T, q_dim]; lse: natural-log softmax denominators [b, n_q, S] fp32.
hipError_t attn_fwd(int dt, const void* qkv, int64_t ld_qkv, void* o, int64_t ld_o, float* lse, int b, int S, int nq,
                    int nkv, int d, hipStream_t st);
// dqkv has the column layout of qkv; delta: workspace for row statistics, [b, n_q, S] fp32 (sums of do*o), for bf16 storage
// twice that; part: workspace of attn_bwd_scratch_floats() floats, or null.  With few KV heads the dK / dV kernel shares the
// query heads of a group out over several workgroups, which leave fp32 partial sums in `part` for a fixed-order reduction; without
// the workspace one workgroup walks the whole group.  cos_tab, sin_tab ([S][d/2] fp32): the q and
// k parts of dqkv come out turned back by the rotary angle of their position, i.e. as gradients w.r.t. the
// projection's output; without them they are gradients w.r.t. the rotated q and k.
size_t attn_bwd_scratch_floats(int dt, int b, int S, int nq, int nkv, int d);
hipError_t attn_bwd(int dt, const void* qkv, int64_t ld_qkv, const void* o, int64_t ld_o, const float* lse,
                    const void* d_o, int64_t ld_do, void* dqkv, int64_t ld_dqkv, float* delta, int b, int S, int nq,
                    int nkv, int d, hipStream_t st, float* part = nullptr, const float* cos_tab = nullptr,
                    const float* sin_tab = nullptr);

// pieces behind the two dispatchers above
hipError_t attn_fwd_f32(const void* qkv, int64_t ld_qkv, void* o, int64_t ld_o, float* lse, int b, int S, int nq, int nkv,
                        int d, hipStream_t st);
size_t attn_bwd_f32_scratch_floats(int b, int S, int nq, int nkv, int d);
hipError_t attn_bwd_f32(const void* qkv, int64_t ld_qkv, const void* o, int64_t ld_o, const float* lse, const void* d_o,
                        int64_t ld_do, void* dqkv, int64_t ld_dqkv, float* delta, int b, int S, int nq, int nkv, int d, hipStream_t st, float* part,
                        const float* cos_tab, const float* sin_tab);
bool bwd_f32_together(int b, int S, int nq, int nkv, int d);  // whether its dQ, dK and dV share a launch.  Host only.
hipError_t attn_fwd_bf16(const void* qkv, int64_t ld_qkv, void* o, int64_t ld_o, float* lse, int b, int S, int nq, int nkv,
                         int d, hipStream_t st);
hipError_t attn_bwd_bf16(const void* qkv, int64_t ld_qkv, const void* o, int64_t ld_o, const float* lse, const void* d_o,
                         int64_t ld_do, void* dqkv, int64_t ld_dqkv, float* stats, int b, int S, int nq, int nkv, int d,
                         hipStream_t st, float* part, const float* cos_tab, const float* sin_tab);

}  // namespace mls
