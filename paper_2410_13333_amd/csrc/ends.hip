// First/last-stage layers (include/mls_ends.h): token embedding gather and its deterministic scatter-add backward;
// final RMSNorm, LM head and mean cross-entropy with the logits gradient formed in place of the logits.  The
// contractions and the RMSNorm are the kernels of the decoder stage; the kernels here are the HBM-bound rest.
#include <hip/hip_runtime.h>

#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/mls.h"
#include "../../include/mls_ends.h"
#include "common.h"
#include "kernels.h"

namespace {

constexpr int TH = 256;
constexpr int MAX_MB = 16;  // micro-batches one scatter launch covers

// ---- x[t, :] = embed[tokens[t], :] (zero row for an id outside the table); one thread per 8 columns.  The thread of a
// row's first columns also keeps the id for the backward (a copy of its own cost 4.5 us per micro-batch beside 15).
template <typename T>
__global__ __launch_bounds__(TH) void embed_gather_kernel(const int32_t* __restrict__ tok, int32_t* __restrict__ keep,
                                                          const T* __restrict__ E, int64_t ld_e, T* __restrict__ x,
                                                          int64_t total, int h, int V) {
  const int64_t id = int64_t(blockIdx.x) * TH + threadIdx.x;
  if (id >= total) return;
  const int cpr = h >> 3;
  const int64_t t = id / cpr;
  const int c = int(id % cpr) * 8;
  const int v = tok[t];
  if (c == 0) keep[t] = v;
  float val[8];
  if (v >= 0 && v < V) {
    load8(E + int64_t(v) * ld_e + c, val);
  } else {
#pragma unroll
    for (int e = 0; e < 8; e++) val[e] = 0.f;
  }
  store8(x + t * h + c, val);
}

// ---- grads_embed[v, :] += sum of the dX rows at the positions that hold token v, in ascending (micro-batch,
// position) order.
// HBM-bound: dX once, and the fp32 rows that some position names read and written.  A workgroup owns up to SC_ROWS table
// rows, 2^shift apart (frequent ids are often neighbours), and a slice of 2048 columns.  It scans the token ids of all
// micro-batches (64 KB from L2 at 16384 positions; one row per workgroup read 2 GB of ids for 32000 rows) and keeps the
// matches as (row, position) keys in LDS, in the order of the positions: ballots count them.  Then the list is split by
// rows, and every thread walks a row's positions for its own eight columns, requesting up to SC_AHEAD rows of dX at a time.
// If the matches do not fit the list, the rows are taken one after the other, each with a scan of its own; a row's sum
// stays in registers all the while, so that it does not depend on which way it came.  Bitwise reproducible, no atomics.
// Measured with the gathers before it (us; one row per workgroup -> 16 neighbouring rows and a list sorted key against key ->
// this): 32000 x 4096, 4 x 4096 uniform ids 606 -> 196 -> 193; ids by Zipf's law 1450 -> 3990 -> 295; half of them one id 7850
// -> 6650 -> 1160; 512 x 256, 4 x 8192 uniform ids 90 -> 530 -> 35; 50304 x 768, 1024 ids 53 -> 9.4 -> 11.5.
struct TokPtrs { const int32_t* p[MAX_MB]; };
// eight elements of a row as they were loaded
template <typename T> struct Chunk8;
template <> struct Chunk8<bf16_t> {
  uint4 r;
  __device__ __forceinline__ void load(const bf16_t* p) { r = *reinterpret_cast<const uint4*>(p); }
  __device__ __forceinline__ void get(float (&v)[8]) const { load8(reinterpret_cast<const bf16_t*>(&r), v); }
};
template <> struct Chunk8<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) { a = reinterpret_cast<const float4*>(p)[0]; b = reinterpret_cast<const float4*>(p)[1]; }
  __device__ __forceinline__ void get(float (&v)[8]) const {
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
};
constexpr int SC_ROWS = 16;    // 4 bits of a key, 28 hold MAX_MB * 2^24 positions
constexpr int SC_CAP = 2048;   // keys of the list (twice 8 KiB of LDS)
constexpr int SC_SCAN = 8;     // ids per thread between two looks at the list's length
static_assert(SC_SCAN * TH <= SC_CAP);
constexpr int SC_AHEAD = 8;
constexpr int SC_GRID = 1024;  // workgroups from which on the rows of one are not made fewer
template <typename T>
__global__ __launch_bounds__(TH) void embed_scatter_kernel(TokPtrs tp, int n, const T* __restrict__ dX, int Ttok, int h,
                                                           int V, int shift, float* __restrict__ gE) {
  constexpr int NW = TH / 64;
  __shared__ uint32_t key[SC_CAP], sorted[SC_CAP];
  __shared__ int found[2][NW], per_row[SC_ROWS];
  const int g0 = blockIdx.x, rows = (V - g0 + (1 << shift) - 1) >> shift;
  const int c = (blockIdx.y * TH + threadIdx.x) * 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t below = (uint64_t(1) << lane) - 1;
  const bool mine = c < h;

  // acc += the dX rows at the first `got` of N positions, in order.  All N are requested (those from `got` on name a valid row,
  // too): with a condition around each, the compiler waits for every one before it requests the next.
  auto add_rows = [&](auto N, const uint32_t (&pos)[SC_AHEAD], int got, float (&acc)[8]) {
    constexpr int some = decltype(N)::value;
    if (!mine) return;
    Chunk8<T> d[some];
#pragma unroll
    for (int q = 0; q < some; q++) d[q].load(dX + int64_t(pos[q]) * h + c);
#pragma unroll
    for (int q = 0; q < some; q++) {
      float v[8];
      d[q].get(v);
#pragma unroll
      for (int e = 0; e < 8; e++) acc[e] = q < got ? acc[e] + v[e] : acc[e];
    }
  };
  using One = std::integral_constant<int, 1>;
  using Ahead = std::integral_constant<int, SC_AHEAD>;
  auto walk = [&](const uint32_t* list, int i0, int i1, float (&acc)[8]) {  // ... at positions list[i0 .. i1)
    for (int at = i0; at < i1; at += SC_AHEAD) {
      uint32_t pos[SC_AHEAD];
#pragma unroll
      for (int q = 0; q < SC_AHEAD; q++) pos[q] = list[min(at + q, i1 - 1)] & 0x0fffffffu;
      add_rows(Ahead{}, pos, min(SC_AHEAD, i1 - at), acc);
    }
  };
  auto add_to_row = [&](int row, const float (&acc)[8]) {
    if (!mine) return;
    float* p = gE + (int64_t(g0) + (int64_t(row) << shift)) * h + c;
    float g[8];
    load8(p, g);
#pragma unroll
    for (int e = 0; e < 8; e++) g[e] += acc[e];
    store8(p, g);
  };
  // Appends the keys that match(id) holds for to the list, ascending in position.  Where the next ones do not fit, full(L) is
  // called first (by the whole workgroup, all keys published); it empties the list (true) or gives up.  Returns the length,
  // or -1.  A wavefront takes SC_SCAN * 64 ids in a row, so that one count per wavefront tells where its keys go.
  auto scan = [&](auto&& match, auto&& full) {
    int L = 0, turn = 0;
    for (int mb = 0; mb < n; mb++) {
      const int32_t* tok = tp.p[mb];
      for (int base = 0; base < Ttok; base += SC_SCAN * TH) {
        const int first = base + wave * (SC_SCAN * 64) + lane;
        int t[SC_SCAN], hits = 0;
        uint64_t hit[SC_SCAN];
#pragma unroll
        for (int q = 0; q < SC_SCAN; q++) t[q] = first + q * 64 < Ttok ? tok[first + q * 64] : -1;
#pragma unroll
        for (int q = 0; q < SC_SCAN; q++) {
          hit[q] = __ballot(match(t[q]));
          hits += __popcll(hit[q]);
        }
        if (lane == 0) found[turn][wave] = hits;
        __syncthreads();  // (the next counts go to the other half: one barrier is enough)
        int at = L, total = 0;
#pragma unroll
        for (int w = 0; w < NW; w++) {
          at += w < wave ? found[turn][w] : 0;
          total += found[turn][w];
        }
        turn ^= 1;
        if (total == 0) continue;
        if (L + total > SC_CAP) {
          if (!full(L)) return -1;
          at -= L;
          L = 0;
        }
        if (hits > 0) {
#pragma unroll
          for (int q = 0; q < SC_SCAN; q++) {
            if (hit[q] >> lane & 1)
              key[at + __popcll(hit[q] & below)] = uint32_t(t[q] >> shift) << 28 | uint32_t(mb * Ttok + first + q * 64);
            at += __popcll(hit[q]);
          }
        }
        L += total;
      }
    }
    __syncthreads();
    return L;
  };

  const int L = rows == 1 ? -1 : scan([&](int t) { return (t & ((1 << shift) - 1)) == g0 && uint32_t(t) < uint32_t(V); },
                                      [](int) { return false; });
  if (L > 0 && L <= 64) {  // a key per lane: the keys of a row are the bits of a mask
    const uint32_t k = lane < L ? key[lane] : 0;
    uint64_t rest = __ballot(lane < L);
    while (rest) {
      const uint32_t row = uint32_t(__builtin_amdgcn_readlane(int(k), __ffsll((unsigned long long)rest) - 1)) >> 28;
      uint64_t m = __ballot(k >> 28 == row) & rest;
      rest &= ~m;
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      while (m) {
        uint32_t pos[SC_AHEAD] = {};  // (read by all lanes, also those without columns)
        int got = 0;
#pragma unroll
        for (int q = 0; q < SC_AHEAD; q++) {
          pos[q] = m ? uint32_t(__builtin_amdgcn_readlane(int(k), __ffsll((unsigned long long)m) - 1)) & 0x0fffffffu : pos[q ? q - 1 : 0];
          got += m ? 1 : 0;
          m &= m - 1;
        }
        if (got == 1) add_rows(One{}, pos, got, acc);
        else add_rows(Ahead{}, pos, got, acc);
      }
      add_to_row(int(row), acc);
    }
  } else if (L > 0) {  // the keys of row r go to sorted[] behind those of the rows before it, in the same order
    for (int r = wave; r < rows; r += NW) {
      int m = 0;
      for (int i = 0; i < L; i += 64) m += __popcll(__ballot(i + lane < L && key[i + lane] >> 28 == uint32_t(r)));
      if (lane == 0) per_row[r] = m;
    }
    __syncthreads();
    for (int r = wave; r < rows; r += NW) {
      if (per_row[r] == 0) continue;
      int at = 0;
      for (int i = 0; i < r; i++) at += per_row[i];
      for (int i = 0; i < L; i += 64) {
        const uint32_t k = i + lane < L ? key[i + lane] : 0;
        const bool it = i + lane < L && k >> 28 == uint32_t(r);
        const uint64_t m = __ballot(it);
        if (it) sorted[at + __popcll(m & below)] = k;
        at += __popcll(m);
      }
    }
    __syncthreads();
    for (int r = 0, at = 0; r < rows; at += per_row[r++]) {
      if (per_row[r] == 0) continue;
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      walk(sorted, at, at + per_row[r], acc);
      add_to_row(r, acc);
    }
  } else if (L < 0) {
    for (int r = 0; r < rows; r++) {
      __syncthreads();  // the list is free
      const int v = g0 + (r << shift);
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      bool any = false;
      const int rest = scan([&](int t) { return t == v; }, [&](int m) {
        any = true;
        __syncthreads();
        walk(key, 0, m, acc);
        __syncthreads();
        return true;
      });
      walk(key, 0, rest, acc);
      if (any || rest > 0) add_to_row(r, acc);
    }
  }
}

// Table rows of a workgroup of the kernel above: 2^shift workgroups share a column slice.  At most SC_ROWS rows each, fewer
// while the grid leaves CUs idle (32 workgroups instead of 512 made most of the 530 us above).
int scatter_shift(int V, int slices) {
  int shift = 0;
  while ((int64_t(SC_ROWS) << shift) < V) shift++;
  while ((int64_t(slices) << shift) < SC_GRID && (1 << shift) < V) shift++;
  return shift;
}

// ---- cross-entropy of one row of logits per workgroup, and its gradient in place:
//   pass 1 (from HBM): running maximum and sum of exponentials per thread, merged across the workgroup;
//   pass 2 (the row is 64 KB or so: from L2): logits <- scale * (exp(logit - lse) - [column == target]).
// An ignored target (outside [0, V)) gives loss 0 and a zero row.
template <typename T>
__global__ __launch_bounds__(TH) void ce_kernel(T* __restrict__ logits, int64_t ld, const int32_t* __restrict__ targets,
                                                int V, float scale, float* __restrict__ row_loss) {
  __shared__ float sm[TH / 64], ss[TH / 64];
  __shared__ float s_lse;
  const int64_t t = blockIdx.x;
  T* row = logits + t * ld;
  const int tgt = targets[t];
  const bool valid = tgt >= 0 && tgt < V;
  const int cpr = V >> 3;
  float m = -INFINITY, s = 0.f;
  for (int c = threadIdx.x; c < cpr; c += TH) {
    float x[8];
    load8(row + c * 8, x);
    float cm = x[0];
#pragma unroll
    for (int e = 1; e < 8; e++) cm = fmaxf(cm, x[e]);
    const float nm = fmaxf(m, cm);
    float add = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e++) add += __expf(x[e] - nm);
    s = s * __expf(m - nm) + add;  // exp(-inf) = 0 on the first chunk
    m = nm;
  }
  // merge (m, s) pairs: lanes, then wavefronts
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float om = __shfl_xor(m, o, 64), os = __shfl_xor(s, o, 64);
    const float nm = fmaxf(m, om);
    s = (m == -INFINITY ? 0.f : s * __expf(m - nm)) + (om == -INFINITY ? 0.f : os * __expf(om - nm));
    m = nm;
  }
  if ((threadIdx.x & 63) == 0) {
    sm[threadIdx.x >> 6] = m;
    ss[threadIdx.x >> 6] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float M = sm[0], S = ss[0];
#pragma unroll
    for (int w = 1; w < TH / 64; w++) {
      const float nm = fmaxf(M, sm[w]);
      S = (M == -INFINITY ? 0.f : S * __expf(M - nm)) + (sm[w] == -INFINITY ? 0.f : ss[w] * __expf(sm[w] - nm));
      M = nm;
    }
    const float lse = M + logf(S);
    s_lse = lse;
    row_loss[t] = valid ? lse - to_f32(row[tgt]) : 0.f;  // read before pass 2 overwrites the row
  }
  __syncthreads();
  const float lse = s_lse;
  for (int c = threadIdx.x; c < cpr; c += TH) {
    float x[8], g[8];
    load8(row + c * 8, x);
#pragma unroll
    for (int e = 0; e < 8; e++) g[e] = valid ? scale * (__expf(x[e] - lse) - (c * 8 + e == tgt ? 1.f : 0.f)) : 0.f;
    store8(row + c * 8, g);
  }
}

// ---- out[0] = (sum of v[0..n)) / n, one workgroup, fixed summation tree
__global__ __launch_bounds__(1024) void mean_kernel(const float* __restrict__ v, int n, float* __restrict__ out) {
  __shared__ float red[16];
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += 1024) s += v[i];
  s = block_sum(s, red);
  if (threadIdx.x == 0) out[0] = s / (float)n;
}

inline int blocks_for(int64_t n) { return int((n + TH - 1) / TH); }
size_t align256(size_t v) { return (v + 255) & ~size_t(255); }
// Row strides as in a stage: the columns from n on, up to whole 64-deep k-tiles, are zero and may be contracted over.
int64_t depth64(int64_t n) { return (n + 63) / 64 * 64; }
int64_t padded(int64_t n, int dt) {
  if (dt == mls::DT_BF16) n = depth64(n);  // (no fp32 kernel reads them)
  return n % 256 == 0 ? n + 64 : n;
}

}  // namespace

// ---- Scratch of mls_head_forward_static: the per-token loss terms between the cross-entropy kernel and the mean.
// One array per GPU (every device that loads this code object holds its own copy until the process ends).  In host
// code the array's name is only a handle for hipGetSymbolAddress; the device address is looked up once per device,
// with that device current, and kernels get that address as an argument.
constexpr int STATIC_TOKENS = 65536;  // 256 KiB
static __device__ __align__(256) float scratch[STATIC_TOKENS];
namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[MAX_DEVICES] = {};
// device address of `scratch` on the current device (looked up on first use there)
hipError_t scratch_address(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    float* p = nullptr;
    if ((e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

struct mls_ends {
  mls_ends_config c;
  int dt, es, T;
  hipStream_t st;
  int64_t ld_h, ld_v;
  size_t off_e, off_g, off_w, n_params;  // public offsets (= layout of grads)
  char *embed = nullptr, *gamma = nullptr, *wlm = nullptr;  // internal: embed [V, ld_h], gamma [h], w_lm [h, ld_v]
  // bf16 storage: w_lm transposed, [V, ld_h], for the forward product (both operands stored along the contraction
  // index is the fastest form of the bf16 GEMM); rewritten whenever the parameters are set
  char* wlm_t = nullptr;
  int32_t* tok = nullptr;  // [max_inflight, T]
  int e_head = 0, e_count = 0;
  // head stash, one entry per kept micro-batch
  char *y = nullptr, *nrm = nullptr, *dlog = nullptr;
  float* r = nullptr;
  size_t mb_h = 0, mb_v = 0;
  int h_head = 0, h_count = 0;
  // workspace
  char* dn = nullptr;
  float *partial = nullptr, *row_loss = nullptr;
  void* split_mem = nullptr;
  mls::SplitSpace split;  // (split_mem) of the products whose contraction is shared out over several workgroups per tile
};

namespace {

int fail(int code, const std::string& msg) { return mls::set_error(code, msg.c_str()); }
int fail_hip(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? MLS_E_NOMEM : MLS_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}
#define HIP_TRY(expr)                                   \
  do {                                                  \
    hipError_t e_ = (expr);                             \
    if (e_ != hipSuccess) return fail_hip(e_, #expr);   \
  } while (0)

hipError_t copy2d(const mls_ends* s, void* dst, int64_t ld_dst, const void* src, int64_t ld_src, int64_t rows,
                  int64_t cols) {
  return hipMemcpy2DAsync(dst, size_t(ld_dst) * s->es, src, size_t(ld_src) * s->es, size_t(cols) * s->es, size_t(rows),
                          hipMemcpyDeviceToDevice, s->st);
}

hipError_t gemm(const mls_ends* s, int mode, const void* A, const void* B, void* C, int M, int N, int K, int64_t lda,
                int64_t ldb, int64_t ldc) {
  return s->dt == mls::DT_BF16 ? mls::gemm_bf16(mode, A, B, C, nullptr, M, N, K, lda, ldb, ldc, 0, s->st, s->split)
                               : mls::gemm_f32(mode, A, B, C, nullptr, M, N, K, lda, ldb, ldc, 0, s->st);
}

void release(mls_ends* s) {
  void* p[] = {s->embed, s->gamma, s->wlm, s->wlm_t, s->tok, s->y, s->nrm, s->dlog, s->r, s->dn, s->partial, s->row_loss,
               s->split_mem};
  for (void* q : p)
    if (q) (void)hipFree(q);
  delete s;
}

// the three parameter tensors: public offset, internal pointer, rows, cols, internal row stride, generator id
struct PT { size_t off; char* ptr; int64_t rows, cols, ld; uint32_t tid; double scale, offset; };
void param_tensors(const mls_ends* s, PT (&t)[3]) {
  const int64_t h = s->c.hidden, V = s->c.vocab;
  t[0] = {s->off_e, s->embed, V, h, s->ld_h, 6, 0.02, 0.0};
  t[1] = {s->off_g, s->gamma, 1, h, h, 7, 0.02, 1.0};
  t[2] = {s->off_w, s->wlm, h, V, s->ld_v, 8, 0.02, 0.0};
}

// the transposed copy of w_lm from w_lm (bf16 storage)
hipError_t transpose_wlm(mls_ends* s) {
  const mls::Spread m = {s->wlm, s->ld_v, nullptr, 0, s->wlm_t, s->ld_h, s->c.hidden, s->c.vocab, 0};
  return mls::spread_bf16(&m, 1, s->st);
}

}  // namespace

extern "C" {

int mls_ends_init(const mls_ends_config* cfg, uint64_t seed, void* hip_stream, mls_ends** out) {
  if (!cfg || !out) return fail(MLS_E_NULL, "mls_ends_init: null argument");
  *out = nullptr;
  const mls_ends_config& c = *cfg;
  if (c.dtype != MLS_BF16 && c.dtype != MLS_FP32) return fail(MLS_E_CONFIG, "dtype must be MLS_BF16 or MLS_FP32");
  if (c.hidden < 8 || c.hidden % 8 || c.hidden > 16384) return fail(MLS_E_CONFIG, "hidden must be a multiple of 8 in [8, 16384]");
  if (c.vocab < 8 || c.vocab % 8) return fail(MLS_E_CONFIG, "vocab must be a positive multiple of 8");
  if (c.seq < 1 || c.micro_batch < 1 || c.max_inflight < 1) return fail(MLS_E_CONFIG, "seq, micro_batch and max_inflight must be positive");
  if (!(c.rms_eps >= 0.f)) return fail(MLS_E_CONFIG, "rms_eps >= 0 required");
  const int64_t T = int64_t(c.seq) * c.micro_batch;
  if (T > (1 << 24) || c.vocab > (1 << 24) || T * int64_t(c.vocab) > (int64_t(1) << 40))
    return fail(MLS_E_CONFIG, "tokens per micro-batch or vocabulary too large");
  mls_ends* s = new mls_ends();
  s->c = c;
  s->dt = c.dtype == MLS_BF16 ? mls::DT_BF16 : mls::DT_FP32;
  s->es = c.dtype == MLS_BF16 ? 2 : 4;
  s->T = int(T);
  s->st = (hipStream_t)hip_stream;
  s->ld_h = padded(c.hidden, s->dt);
  s->ld_v = padded(c.vocab, s->dt);
  const size_t h = c.hidden, V = c.vocab;
  s->off_e = 0;
  s->off_g = V * h;
  s->off_w = s->off_g + h;
  s->n_params = s->off_w + h * V;
  s->mb_h = align256(size_t(T) * s->ld_h * s->es);
  s->mb_v = align256(size_t(T) * s->ld_v * s->es);
  const size_t nmb = c.max_inflight;
  const size_t split = s->dt != mls::DT_BF16 ? 0 :
      mls::split_bytes(std::max(mls::gemm_split_floats(mls::T16_NT, s->T, int(V), int(depth64(h))),
                                mls::gemm_split_floats(mls::T16_NT, s->T, int(h), int(depth64(V)))));
  auto alloc = [&](void** p, size_t bytes) { return hipMalloc(p, bytes ? bytes : 256); };
  hipError_t e = hipSuccess;
  if ((e = alloc((void**)&s->embed, V * s->ld_h * s->es)) != hipSuccess ||
      (e = alloc((void**)&s->gamma, h * s->es)) != hipSuccess ||
      (e = alloc((void**)&s->wlm, h * s->ld_v * s->es)) != hipSuccess ||
      (s->dt == mls::DT_BF16 && (e = alloc((void**)&s->wlm_t, V * s->ld_h * s->es)) != hipSuccess) ||
      (e = alloc((void**)&s->tok, nmb * T * 4)) != hipSuccess ||
      (e = alloc((void**)&s->y, nmb * s->mb_h)) != hipSuccess ||
      (e = alloc((void**)&s->nrm, nmb * s->mb_h)) != hipSuccess ||
      (e = alloc((void**)&s->dlog, nmb * s->mb_v)) != hipSuccess ||
      (e = alloc((void**)&s->r, nmb * T * 4)) != hipSuccess ||
      (e = alloc((void**)&s->dn, s->mb_h)) != hipSuccess ||
      (e = alloc((void**)&s->partial, size_t(mls::rmsnorm_bwd_blocks(s->T)) * h * 4)) != hipSuccess ||
      (e = alloc((void**)&s->row_loss, T * 4)) != hipSuccess ||
      (split && (e = alloc(&s->split_mem, split)) != hipSuccess)) {
    release(s);
    return fail_hip(e, "hipMalloc");
  }
  if (s->dt == mls::DT_BF16 && (h % 64 || V % 64)) {
    if ((e = hipMemsetAsync(s->wlm, 0, h * s->ld_v * s->es, s->st)) != hipSuccess ||
        (e = hipMemsetAsync(s->wlm_t, 0, V * s->ld_h * s->es, s->st)) != hipSuccess ||
        (e = hipMemsetAsync(s->nrm, 0, nmb * s->mb_h, s->st)) != hipSuccess ||
        (e = hipMemsetAsync(s->dlog, 0, nmb * s->mb_v, s->st)) != hipSuccess) {
      release(s);
      return fail_hip(e, "hipMemsetAsync");
    }
  }
  s->split = mls::split_space(s->split_mem);
  if (split && (e = hipMemsetAsync(s->split.state, 0, size_t(mls::SPLIT_TILES) * 8, s->st)) != hipSuccess) {
    release(s);
    return fail_hip(e, "hipMemsetAsync");
  }
  PT t[3];
  param_tensors(s, t);
  for (auto& q : t)
    if ((e = mls::fill_normal(s->dt, q.ptr, q.rows, q.cols, q.ld, seed, q.tid, 0, q.scale, q.offset, s->st)) != hipSuccess) {
      release(s);
      return fail_hip(e, "weight generator");
    }
  if (s->wlm_t && (e = transpose_wlm(s)) != hipSuccess) {
    release(s);
    return fail_hip(e, "spread_bf16");
  }
  if ((e = hipStreamSynchronize(s->st)) != hipSuccess) {
    release(s);
    return fail_hip(e, "hipStreamSynchronize");
  }
  float* sp = nullptr;  // set-up of mls_head_forward_static on this device
  if ((e = scratch_address(&sp)) != hipSuccess) {
    release(s);
    return fail_hip(e, "hipGetSymbolAddress(scratch)");
  }
  *out = s;
  return MLS_OK;
}

void mls_ends_free(mls_ends* s) {
  if (!s) return;
  (void)hipStreamSynchronize(s->st);
  release(s);
}

int mls_embed_forward(mls_ends* s, const int32_t* tokens, void* x) {
  if (!s || !tokens || !x) return fail(MLS_E_NULL, "mls_embed_forward: null argument");
  if ((uintptr_t(tokens) & 3) || (uintptr_t(x) & 15)) return fail(MLS_E_CONFIG, "mls_embed_forward: x must be 16-byte aligned");
  if (s->e_count >= s->c.max_inflight) return fail(MLS_E_STASH, "embedding stash full: max_inflight micro-batches already forwarded");
  const int slot = (s->e_head + s->e_count) % s->c.max_inflight;
  int32_t* keep = s->tok + size_t(slot) * s->T;
  const int64_t total = int64_t(s->T) * (s->c.hidden >> 3);
  if (s->dt == mls::DT_BF16)
    hipLaunchKernelGGL(embed_gather_kernel<bf16_t>, dim3(blocks_for(total)), dim3(TH), 0, s->st, tokens, keep,
                       (const bf16_t*)s->embed, s->ld_h, (bf16_t*)x, total, s->c.hidden, s->c.vocab);
  else
    hipLaunchKernelGGL(embed_gather_kernel<float>, dim3(blocks_for(total)), dim3(TH), 0, s->st, tokens, keep,
                       (const float*)s->embed, s->ld_h, (float*)x, total, s->c.hidden, s->c.vocab);
  HIP_TRY(hipGetLastError());
  s->e_count++;
  return MLS_OK;
}

int mls_embed_backward(mls_ends* s, const void* dX, float* grads, int32_t n) {
  if (!s) return fail(MLS_E_NULL, "mls_embed_backward: null handle");
  if (n < 0) return fail(MLS_E_RANGE, "n_microbatches must be >= 0");
  if (n == 0) return MLS_OK;
  if (!dX || !grads) return fail(MLS_E_NULL, "mls_embed_backward: null argument");
  if ((uintptr_t(dX) | uintptr_t(grads)) & 15) return fail(MLS_E_CONFIG, "mls_embed_backward: dX and grads must be 16-byte aligned");
  if (n > s->e_count) return fail(MLS_E_STASH, "n_microbatches exceeds the kept embedding micro-batches");
  const int h = s->c.hidden;
  const size_t act = size_t(s->T) * h * s->es;
  for (int i0 = 0; i0 < n; i0 += MAX_MB) {
    const int m = n - i0 < MAX_MB ? n - i0 : MAX_MB;
    TokPtrs tp = {};
    for (int i = 0; i < m; i++) tp.p[i] = s->tok + size_t((s->e_head + i0 + i) % s->c.max_inflight) * s->T;
    const char* dx = (const char*)dX + size_t(i0) * act;
    float* gE = grads + s->off_e;
    const int slices = (h / 8 + TH - 1) / TH, shift = scatter_shift(s->c.vocab, slices);
#define SCATTER(TY)                                                                                                  \
  hipLaunchKernelGGL(embed_scatter_kernel<TY>, dim3(std::min(1 << shift, s->c.vocab), slices), dim3(TH), 0, s->st, tp, m, \
                     (const TY*)dx, s->T, h, s->c.vocab, shift, gE)
    if (s->dt == mls::DT_BF16) SCATTER(bf16_t); else SCATTER(float);
#undef SCATTER
    HIP_TRY(hipGetLastError());
  }
  s->e_head = (s->e_head + n) % s->c.max_inflight;
  s->e_count -= n;
  return MLS_OK;
}

// row_loss: T floats of scratch for the per-token loss terms (every one is written before the mean reads it)
static int head_forward(mls_ends* s, const void* y, const int32_t* targets, float loss_weight, float* loss, float* row_loss) {
  if (s->h_count >= s->c.max_inflight) return fail(MLS_E_STASH, "head stash full: max_inflight micro-batches already forwarded");
  const int slot = (s->h_head + s->h_count) % s->c.max_inflight;
  const int T = s->T, h = s->c.hidden, V = s->c.vocab;
  char* ys = s->y + size_t(slot) * s->mb_h;
  char* nr = s->nrm + size_t(slot) * s->mb_h;
  char* dl = s->dlog + size_t(slot) * s->mb_v;
  float* r = s->r + size_t(slot) * T;
  HIP_TRY(mls::rmsnorm_fwd(s->dt, y, h, s->gamma, nr, s->ld_h, r, T, h, s->c.rms_eps, s->st, ys, s->ld_h));
  if (s->wlm_t) HIP_TRY(gemm(s, mls::GEMM_NT, nr, s->wlm_t, dl, T, V, int(depth64(h)), s->ld_h, s->ld_h, s->ld_v));
  else HIP_TRY(gemm(s, mls::GEMM_NN, nr, s->wlm, dl, T, V, h, s->ld_h, s->ld_v, s->ld_v));
  const float scale = loss_weight / (float)T;
  if (s->dt == mls::DT_BF16)
    hipLaunchKernelGGL(ce_kernel<bf16_t>, dim3(T), dim3(TH), 0, s->st, (bf16_t*)dl, s->ld_v, targets, V, scale, row_loss);
  else
    hipLaunchKernelGGL(ce_kernel<float>, dim3(T), dim3(TH), 0, s->st, (float*)dl, s->ld_v, targets, V, scale, row_loss);
  HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(1024), 0, s->st, row_loss, T, loss);
  HIP_TRY(hipGetLastError());
  s->h_count++;
  return MLS_OK;
}

int mls_head_forward(mls_ends* s, const void* y, const int32_t* targets, float loss_weight, float* loss) {
  if (!s || !y || !targets || !loss) return fail(MLS_E_NULL, "mls_head_forward: null argument");
  if (uintptr_t(y) & 15) return fail(MLS_E_CONFIG, "mls_head_forward: y must be 16-byte aligned");
  return head_forward(s, y, targets, loss_weight, loss, s->row_loss);
}

int mls_head_forward_static(mls_ends* s, const void* y, const int32_t* targets, float loss_weight, float* loss) {
  if (!s || !y || !targets || !loss) return fail(MLS_E_NULL, "mls_head_forward_static: null argument");
  if (uintptr_t(y) & 15) return fail(MLS_E_CONFIG, "mls_head_forward_static: y must be 16-byte aligned");
  if (s->T > STATIC_TOKENS)
    return fail(MLS_E_RANGE, "mls_head_forward_static: more than 65536 tokens per micro-batch (the static scratch holds 65536 loss terms)");
  float* sp = nullptr;
  if (hipError_t e = scratch_address(&sp)) return fail_hip(e, "hipGetSymbolAddress(scratch)");
  return head_forward(s, y, targets, loss_weight, loss, sp);
}

int mls_head_backward(mls_ends* s, float* grads, int32_t n, void* dY) {
  if (!s) return fail(MLS_E_NULL, "mls_head_backward: null handle");
  if (n < 0) return fail(MLS_E_RANGE, "n_microbatches must be >= 0");
  if (n == 0) return MLS_OK;
  if (!grads || !dY) return fail(MLS_E_NULL, "mls_head_backward: null argument");
  if ((uintptr_t(dY) | uintptr_t(grads)) & 15) return fail(MLS_E_CONFIG, "mls_head_backward: dY and grads must be 16-byte aligned");
  if (n > s->h_count) return fail(MLS_E_STASH, "n_microbatches exceeds the kept head micro-batches");
  const int T = s->T, h = s->c.hidden, V = s->c.vocab;
  const size_t act = size_t(T) * h * s->es;
  std::vector<const void*> an, bd;
  for (int i = 0; i < n; i++) {
    const int slot = (s->h_head + i) % s->c.max_inflight;
    const char* ys = s->y + size_t(slot) * s->mb_h;
    const char* nr = s->nrm + size_t(slot) * s->mb_h;
    const char* dl = s->dlog + size_t(slot) * s->mb_v;
    const float* r = s->r + size_t(slot) * T;
    // d nrm = dlogits w_lm^T; then the RMSNorm backward straight into the caller's dY
    HIP_TRY(gemm(s, mls::GEMM_NT, dl, s->wlm, s->dn, T, h, s->dt == mls::DT_BF16 ? int(depth64(V)) : V, s->ld_v, s->ld_v, s->ld_h));
    HIP_TRY(mls::rmsnorm_bwd(s->dt, s->dn, s->ld_h, ys, s->ld_h, s->gamma, r, nullptr, 0, (char*)dY + size_t(i) * act, h,
                             grads + s->off_g, s->partial, T, h, s->st));
    an.push_back(nr);
    bd.push_back(dl);
  }
  // grads_w_lm += sum_i nrm_i^T dlogits_i: one contraction over all micro-batches where the DMA path can
  float* gw = grads + s->off_w;
  if (s->dt == mls::DT_BF16 && mls::gemm_tn_segments_ok(T, s->ld_h, s->ld_v)) {
    for (int i = 0; i < n; i += 16)
      HIP_TRY(mls::gemm_bf16_tn_segments(an.data() + i, bd.data() + i, n - i < 16 ? n - i : 16, gw, h, V, T, s->ld_h, s->ld_v, V, s->st));
  } else {
    for (int i = 0; i < n; i++) HIP_TRY(gemm(s, mls::GEMM_TN, an[i], bd[i], gw, h, V, T, s->ld_h, s->ld_v, V));
  }
  s->h_head = (s->h_head + n) % s->c.max_inflight;
  s->h_count -= n;
  return MLS_OK;
}

size_t mls_ends_grad_elems(const mls_ends* s) { return s ? s->n_params : 0; }

int mls_ends_param_layout(const mls_ends* s, int32_t which, size_t* offset, size_t* rows, size_t* cols) {
  if (!s || !offset || !rows || !cols) return fail(MLS_E_NULL, "mls_ends_param_layout: null argument");
  const size_t h = s->c.hidden, V = s->c.vocab;
  switch (which) {
    case MLS_PE_EMBED: *offset = s->off_e; *rows = V; *cols = h; break;
    case MLS_PE_GAMMA_F: *offset = s->off_g; *rows = 1; *cols = h; break;
    case MLS_PE_WLM: *offset = s->off_w; *rows = h; *cols = V; break;
    default: return fail(MLS_E_RANGE, "unknown parameter id");
  }
  return MLS_OK;
}

int mls_ends_get_params(mls_ends* s, void* dst) {
  if (!s || !dst) return fail(MLS_E_NULL, "mls_ends_get_params: null argument");
  PT t[3];
  param_tensors(s, t);
  for (auto& q : t) HIP_TRY(copy2d(s, (char*)dst + q.off * s->es, q.cols, q.ptr, q.ld, q.rows, q.cols));
  HIP_TRY(hipStreamSynchronize(s->st));
  return MLS_OK;
}

int mls_ends_set_params(mls_ends* s, const void* src) {
  if (!s || !src) return fail(MLS_E_NULL, "mls_ends_set_params: null argument");
  PT t[3];
  param_tensors(s, t);
  if (s->wlm_t && !(uintptr_t(src) & 15)) {  // bf16: all three in one pass, the transposed w_lm with them
    mls::Spread m[3];
    for (int i = 0; i < 3; i++)
      m[i] = {(const char*)src + t[i].off * s->es, t[i].cols, t[i].ptr, t[i].ld, i == 2 ? s->wlm_t : nullptr, s->ld_h,
              int(t[i].rows), int(t[i].cols), 0};
    HIP_TRY(mls::spread_bf16(m, 3, s->st));
  } else {
    for (auto& q : t) HIP_TRY(copy2d(s, q.ptr, q.ld, (const char*)src + q.off * s->es, q.cols, q.rows, q.cols));
    if (s->wlm_t) HIP_TRY(transpose_wlm(s));
  }
  HIP_TRY(hipStreamSynchronize(s->st));
  return MLS_OK;
}

int mls_ends_inflight(const mls_ends* s, int32_t* embed, int32_t* head) {
  if (!s) return fail(MLS_E_NULL, "null handle");
  if (embed) *embed = s->e_count;
  if (head) *head = s->h_count;
  return MLS_OK;
}

int mls_ends_debug_dlogits(mls_ends* s, int32_t slot, void* dst) {
  if (!s || !dst) return fail(MLS_E_NULL, "mls_ends_debug_dlogits: null argument");
  if (slot < 0 || slot >= s->h_count) return fail(MLS_E_RANGE, "head stash slot out of range");
  const int phys = (s->h_head + slot) % s->c.max_inflight;
  HIP_TRY(copy2d(s, dst, s->c.vocab, s->dlog + size_t(phys) * s->mb_v, s->ld_v, s->T, s->c.vocab));
  HIP_TRY(hipStreamSynchronize(s->st));
  return MLS_OK;
}

}  // extern "C"
