// HBM-bound kernels of the decoder layer: RMSNorm forward/backward (with the residual-gradient add fused),
// rotary embedding, SwiGLU forward/backward, and the weight generator.  All use 16-byte accesses, fp32
// arithmetic and wavefront (64-lane) reductions; each tensor is read once and written once.
#include "common.h"
#include "kernels.h"

namespace {

constexpr int EW_THREADS = 256;
// NORM_MAXC = 16-byte chunks per thread a row may span (template argument MAXC of the norm kernels):
// hidden <= MAXC * 8 * 256; instantiated for 2, 4 and 8 so that narrow rows do not pay for wide ones in registers

// ---------------------------------------------------------------- RMSNorm forward: one workgroup per row
// copy (may be null): receives x, row stride ldc, on the way (a caller's dense rows into a padded buffer)
template <typename T, int NORM_MAXC>
__global__ __launch_bounds__(EW_THREADS) void rmsnorm_fwd_kernel(const T* __restrict__ x, int64_t ldx,
                                                                 const T* __restrict__ gamma, T* __restrict__ a,
                                                                 int64_t lda, float* __restrict__ rstd, int h,
                                                                 float eps, T* __restrict__ copy, int64_t ldc) {
  __shared__ float red[EW_THREADS / 64];
  const int64_t row = blockIdx.x;
  const T* xr = x + row * ldx;
  const int nchunk = h >> 3;
  float v[NORM_MAXC][8];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NORM_MAXC; i++) {
    const int c = threadIdx.x + i * EW_THREADS;
    if (c < nchunk) {
      load8(xr + c * 8, v[i]);
      if (copy) store8(copy + row * ldc + c * 8, v[i]);
#pragma unroll
      for (int e = 0; e < 8; e++) ss += v[i][e] * v[i][e];
    }
  }
  const float r = rsqrtf(block_sum(ss, red) / (float)h + eps);
  if (threadIdx.x == 0) rstd[row] = r;
#pragma unroll
  for (int i = 0; i < NORM_MAXC; i++) {
    const int c = threadIdx.x + i * EW_THREADS;
    if (c < nchunk) {
      float g[8], o[8];
      load8(gamma + c * 8, g);
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = v[i][e] * r * g[e];
      store8(a + row * lda + c * 8, o);
    }
  }
}

// ---------------------------------------------------------------- RMSNorm of many narrow rows: one wavefront per row (bf16)
// A workgroup per row leaves half of its threads or more without a chunk and waits for two barriers per row; here a row's sum is a
// wavefront's own.  MAXC: 16-byte chunks per lane.  Both norms of a layer, forward and backward, with the reduction of the gains (us,
// workgroup per row -> wavefront per row): 12288 rows of 256 90 -> 45, 4096 of 512 49 -> 37, 4096 of 1024 53 -> 45, 2048 of 256 37 -> 33.
template <int MAXC>
__global__ __launch_bounds__(EW_THREADS) void rmsnorm_fwd_wave_kernel(const bf16_t* __restrict__ x, int64_t ldx, const bf16_t* __restrict__ gamma,
                                                                      bf16_t* __restrict__ a, int64_t lda, float* __restrict__ rstd, int rows,
                                                                      int h, float eps, bf16_t* __restrict__ copy, int64_t ldc) {
  const int lane = threadIdx.x & 63, nchunk = h >> 3;
  const int64_t row = int64_t(blockIdx.x) * (EW_THREADS / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  float v[MAXC][8], g[MAXC][8], ss = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = lane + i * 64;
    if (c < nchunk) {
      load8(x + row * ldx + c * 8, v[i]);
      load8(gamma + c * 8, g[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = lane + i * 64;
    if (c < nchunk) {
      if (copy) store8(copy + row * ldc + c * 8, v[i]);
#pragma unroll
      for (int e = 0; e < 8; e++) ss += v[i][e] * v[i][e];
    }
  }
  const float r = rsqrtf(wave_sum(ss) / (float)h + eps);
  if (lane == 0) rstd[row] = r;
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = lane + i * 64;
    if (c < nchunk) {
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = v[i][e] * r * g[i][e];
      store8(a + row * lda + c * 8, o);
    }
  }
}

// Wavefront w of workgroup b takes rows 4 b + w, 4 (b + gridDim.x) + w, ...; the four wavefronts' column sums for dgamma meet in
// LDS, in their order, and go to partial[b][:].
template <int MAXC>
__global__ __launch_bounds__(EW_THREADS) void rmsnorm_bwd_wave_kernel(const bf16_t* __restrict__ da, int64_t ld_da, const bf16_t* __restrict__ x,
                                                                      int64_t ldx, const bf16_t* __restrict__ gamma,
                                                                      const float* __restrict__ rstd, const bf16_t* dres, int64_t ld_dres,
                                                                      bf16_t* dx, int64_t ld_dx, float* __restrict__ partial, int rows, int h,
                                                                      bool acc_partial) {
  constexpr int W = EW_THREADS / 64;
  __shared__ float sums[W][MAXC * 512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nchunk = h >> 3;
  float g[MAXC][8], dg[MAXC][8];
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = lane + i * 64;
#pragma unroll
    for (int e = 0; e < 8; e++) dg[i][e] = 0.f;
    if (c < nchunk) load8(gamma + c * 8, g[i]);
  }
  for (int64_t row = int64_t(blockIdx.x) * W + wave; row < rows; row += int64_t(gridDim.x) * W) {
    const float r = rstd[row];
    float n[MAXC][8], dn[MAXC][8], res[MAXC][8], dot = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; i++) {
      const int c = lane + i * 64;
      if (c < nchunk) {
        load8(x + row * ldx + c * 8, n[i]);
        load8(da + row * ld_da + c * 8, dn[i]);
        if (dres) {
          load8(dres + row * ld_dres + c * 8, res[i]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; e++) res[i][e] = 0.f;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < MAXC; i++) {
      const int c = lane + i * 64;
      if (c < nchunk) {
#pragma unroll
        for (int e = 0; e < 8; e++) {
          n[i][e] *= r;
          dg[i][e] += dn[i][e] * n[i][e];
          dn[i][e] *= g[i][e];
          dot += dn[i][e] * n[i][e];
        }
      }
    }
    const float mean = wave_sum(dot) / (float)h;
#pragma unroll
    for (int i = 0; i < MAXC; i++) {
      const int c = lane + i * 64;
      if (c < nchunk) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = res[i][e] + r * (dn[i][e] - n[i][e] * mean);
        store8(dx + row * ld_dx + c * 8, o);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < MAXC; i++)
    if (lane + i * 64 < nchunk) store8(&sums[wave][(lane + i * 64) * 8], dg[i]);
  __syncthreads();
  for (int c = threadIdx.x * 4; c < h; c += EW_THREADS * 4) {
    float4* p = reinterpret_cast<float4*>(partial + int64_t(blockIdx.x) * h + c);
    float4 t = *reinterpret_cast<const float4*>(&sums[0][c]);
#pragma unroll
    for (int w = 1; w < W; w++) {
      const float4 u = *reinterpret_cast<const float4*>(&sums[w][c]);
      t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
    }
    if (acc_partial) {  // on top of what earlier calls left (same workgroup, same rows' share: a fixed order)
      const float4 u = *p;
      t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
    }
    *p = t;
  }
}

// rows of cpr 16-byte chunks; blockIdx.y: one of several matrices, next_* bytes apart
__global__ __launch_bounds__(EW_THREADS) void copy_rows_kernel(const char* __restrict__ src, int64_t ld_src, int64_t next_src,
                                                               char* __restrict__ dst, int64_t ld_dst, int64_t next_dst, int cpr,
                                                               int64_t total) {
  const int64_t id = int64_t(blockIdx.x) * EW_THREADS + threadIdx.x;
  if (id >= total) return;
  const int64_t row = id / cpr, at = (id - row * cpr) * 16;
  *reinterpret_cast<uint4*>(dst + blockIdx.y * next_dst + row * ld_dst + at) =
      *reinterpret_cast<const uint4*>(src + blockIdx.y * next_src + row * ld_src + at);
}

// eight consecutive bf16 elements as they lie in memory (16 bytes), converted on demand
template <typename T>
struct Raw8;
template <>
struct Raw8<bf16_t> {
  uint4 v;
  __device__ __forceinline__ void load(const bf16_t* p) { v = *reinterpret_cast<const uint4*>(p); }
  __device__ __forceinline__ void get(float (&o)[8]) const {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};
// ---------------------------------------------------------------- RMSNorm backward
// Workgroup w handles rows w, w + gridDim.x, ...; it keeps its share of the column sums for dgamma in
// registers and writes them to partial[w][:], which a second kernel adds up in a fixed order.
template <typename T, int NORM_MAXC>
__global__ __launch_bounds__(EW_THREADS) void rmsnorm_bwd_kernel(const T* __restrict__ da, int64_t ld_da,
                                                                 const T* __restrict__ x, int64_t ldx,
                                                                 const T* __restrict__ gamma,
                                                                 const float* __restrict__ rstd, const T* dres,
                                                                 int64_t ld_dres, T* dx, int64_t ld_dx,
                                                                 float* __restrict__ partial, int rows, int h,
                                                                 bool acc_partial) {
  __shared__ float red[EW_THREADS / 64];
  const int nchunk = h >> 3;
  float g[NORM_MAXC][8], dg[NORM_MAXC][8];
#pragma unroll
  for (int i = 0; i < NORM_MAXC; i++) {
    const int c = threadIdx.x + i * EW_THREADS;
#pragma unroll
    for (int e = 0; e < 8; e++) dg[i][e] = 0.f;
    if (c < nchunk) load8(gamma + c * 8, g[i]);
  }
  // bf16 rows of up to 8192 elements are software-pipelined: the (unconverted) operands of the workgroup's next
  // row are requested before the current row is reduced, so that two rows per workgroup are in flight.  Wider or
  // fp32 rows would not fit the registers that way and take the plain loop.
  if constexpr (sizeof(T) == 2 && NORM_MAXC <= 4) {
    Raw8<T> rx[NORM_MAXC], rda[NORM_MAXC], rres[NORM_MAXC];
    auto request = [&](int64_t row) {
#pragma unroll
      for (int i = 0; i < NORM_MAXC; i++) {
        const int c = threadIdx.x + i * EW_THREADS;
        if (c < nchunk) {
          rx[i].load(x + row * ldx + c * 8);
          rda[i].load(da + row * ld_da + c * 8);
          if (dres) rres[i].load(dres + row * ld_dres + c * 8);
        }
      }
    };
    if (blockIdx.x < rows) request(blockIdx.x);
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
      const float r = rstd[row];
      float n[NORM_MAXC][8], dn[NORM_MAXC][8], res[NORM_MAXC][8];
      float dot = 0.f;
#pragma unroll
      for (int i = 0; i < NORM_MAXC; i++) {
        const int c = threadIdx.x + i * EW_THREADS;
        if (c < nchunk) {
          float xv[8], dav[8];
          rx[i].get(xv);
          rda[i].get(dav);
          if (dres) {
            rres[i].get(res[i]);
          } else {
#pragma unroll
            for (int e = 0; e < 8; e++) res[i][e] = 0.f;
          }
#pragma unroll
          for (int e = 0; e < 8; e++) {
            n[i][e] = xv[e] * r;
            dn[i][e] = dav[e] * g[i][e];
            dg[i][e] += dav[e] * n[i][e];
            dot += dn[i][e] * n[i][e];
          }
        }
      }
      if (row + gridDim.x < rows) request(row + gridDim.x);
      const float mean = block_sum(dot, red) / (float)h;
#pragma unroll
      for (int i = 0; i < NORM_MAXC; i++) {
        const int c = threadIdx.x + i * EW_THREADS;
        if (c < nchunk) {
          float o[8];
#pragma unroll
          for (int e = 0; e < 8; e++) o[e] = res[i][e] + r * (dn[i][e] - n[i][e] * mean);
          store8(dx + row * ld_dx + c * 8, o);
        }
      }
    }
  } else {
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
      const float r = rstd[row];
      float n[NORM_MAXC][8], dn[NORM_MAXC][8];
      float dot = 0.f;
#pragma unroll
      for (int i = 0; i < NORM_MAXC; i++) {
        const int c = threadIdx.x + i * EW_THREADS;
        if (c < nchunk) {
          float xv[8], dav[8];
          load8(x + row * ldx + c * 8, xv);
          load8(da + row * ld_da + c * 8, dav);
#pragma unroll
          for (int e = 0; e < 8; e++) {
            n[i][e] = xv[e] * r;
            dn[i][e] = dav[e] * g[i][e];
            dg[i][e] += dav[e] * n[i][e];
            dot += dn[i][e] * n[i][e];
          }
        }
      }
      float res[NORM_MAXC][8];  // requested before the reduction so that their latency overlaps it
#pragma unroll
      for (int i = 0; i < NORM_MAXC; i++) {
        const int c = threadIdx.x + i * EW_THREADS;
        if (c < nchunk) {
          if (dres) {
            load8(dres + row * ld_dres + c * 8, res[i]);
          } else {
#pragma unroll
            for (int e = 0; e < 8; e++) res[i][e] = 0.f;
          }
        }
      }
      const float mean = block_sum(dot, red) / (float)h;
#pragma unroll
      for (int i = 0; i < NORM_MAXC; i++) {
        const int c = threadIdx.x + i * EW_THREADS;
        if (c < nchunk) {
          float o[8];
#pragma unroll
          for (int e = 0; e < 8; e++) o[e] = res[i][e] + r * (dn[i][e] - n[i][e] * mean);
          store8(dx + row * ld_dx + c * 8, o);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NORM_MAXC; i++) {
    const int c = threadIdx.x + i * EW_THREADS;
    if (c < nchunk) {
      float* p = partial + int64_t(blockIdx.x) * h + c * 8;
      if (acc_partial) {  // on top of what earlier calls left (same workgroup, same rows' share: a fixed order)
        float prev[8];
        load8(p, prev);
#pragma unroll
        for (int e = 0; e < 8; e++) dg[i][e] += prev[e];
      }
      store8(p, dg[i]);
    }
  }
}

__global__ __launch_bounds__(256) void colsum_add_kernel(mls::Colsum cs) {
  __shared__ float red[COLSUM_LDS];
  colsum_block(cs, blockIdx.x, red);
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float4* __restrict__ p, size_t n4) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < n4) p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// ---------------------------------------------------------------- rotary embedding, in place (bf16 storage; fp32: in the product before it)
// One thread rotates 8 pairs (i .. i+7, i+d/2 .. i+d/2+7) of one head of one token.
__global__ __launch_bounds__(EW_THREADS) void rope_kernel(bf16_t* __restrict__ u, const float* __restrict__ cos_tab,
                                                          const float* __restrict__ sin_tab, int64_t total, int S,
                                                          int n_heads, int d, int64_t ld) {
  const int64_t id = int64_t(blockIdx.x) * EW_THREADS + threadIdx.x;
  if (id >= total) return;
  const int cph = d >> 4;  // chunks of 8 pairs per head
  const int c = int(id % cph);
  const int head = int((id / cph) % n_heads);
  const int64_t t = id / (int64_t(cph) * n_heads);
  const int pos = int(t % S);
  bf16_t* p = u + t * ld + head * d + c * 8;
  float a[8], b[8], cs[8], sn[8], oa[8], ob[8];
  load8(p, a);
  load8(p + (d >> 1), b);
  load8(cos_tab + int64_t(pos) * (d >> 1) + c * 8, cs);
  load8(sin_tab + int64_t(pos) * (d >> 1) + c * 8, sn);
#pragma unroll
  for (int e = 0; e < 8; e++) {
    oa[e] = a[e] * cs[e] - b[e] * sn[e];
    ob[e] = a[e] * sn[e] + b[e] * cs[e];
  }
  store8(p, oa);
  store8(p + (d >> 1), ob);
}

// ---------------------------------------------------------------- SwiGLU (bf16 storage; fp32: epilogues of the products)

__global__ __launch_bounds__(EW_THREADS) void swiglu_fwd_kernel(const bf16_t* __restrict__ gu, int64_t ld_gu,
                                                                bf16_t* __restrict__ z, int64_t ld_z, int64_t total,
                                                                int f) {
  const int64_t id = int64_t(blockIdx.x) * EW_THREADS + threadIdx.x;
  if (id >= total) return;
  const int cpr = f >> 3;
  const int64_t t = id / cpr;
  const int c = int(id % cpr);
  float g[8], u[8], o[8];
  load8(gu + t * ld_gu + c * 8, g);
  load8(gu + t * ld_gu + f + c * 8, u);
#pragma unroll
  for (int e = 0; e < 8; e++) o[e] = g[e] * sigmoidf_(g[e]) * u[e];
  store8(z + t * ld_z + c * 8, o);
}

// IL: gu and dgu are in the interleaved gate/up column order (32 gates, their 32 ups, ...), else [gates | ups]
template <bool IL>
__global__ __launch_bounds__(EW_THREADS) void swiglu_bwd_kernel(const bf16_t* __restrict__ dz, int64_t ld_dz,
                                                                const bf16_t* __restrict__ gu, int64_t ld_gu,
                                                                bf16_t* __restrict__ dgu, int64_t ld_dgu, int64_t total,
                                                                int f) {
  const int64_t id = int64_t(blockIdx.x) * EW_THREADS + threadIdx.x;
  if (id >= total) return;
  const int cpr = f >> 3;
  const int64_t t = id / cpr;
  const int c = int(id % cpr) * 8;
  const int cg = IL ? (c >> 5) * 64 + (c & 31) : c, cu = IL ? cg + 32 : f + c;
  float g[8], u[8], d[8], og[8], ou[8];
  load8(gu + t * ld_gu + cg, g);
  load8(gu + t * ld_gu + cu, u);
  load8(dz + t * ld_dz + c, d);
#pragma unroll
  for (int e = 0; e < 8; e++) {
    const float s = sigmoidf_(g[e]);
    og[e] = d[e] * u[e] * s * (1.f + g[e] * (1.f - s));
    ou[e] = d[e] * g[e] * s;
  }
  store8(dgu + t * ld_dgu + cg, og);
  store8(dgu + t * ld_dgu + cu, ou);
}

// ---------------------------------------------------------------- weight generator (counter-based, fp64 Box-Muller)
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// fp64 -> bf16 bits, one round-to-nearest-even (normal range)
__device__ __forceinline__ uint16_t f64_to_bf16_bits(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t sign = uint32_t(u >> 63) << 15;
  const int exp = int((u >> 52) & 0x7ff);
  if (exp == 0) return (uint16_t)sign;
  const uint64_t man = u & ((1ull << 52) - 1);
  uint32_t keep = (uint32_t(exp - 1023 + 127) << 7) | uint32_t(man >> 45);
  const uint64_t rem = man & ((1ull << 45) - 1), half = 1ull << 44;
  if (rem > half || (rem == half && (keep & 1))) keep += 1;
  return (uint16_t)(sign | keep);
}
__device__ __forceinline__ void put(bf16_t* p, double v) { *reinterpret_cast<uint16_t*>(p) = f64_to_bf16_bits(v); }
__device__ __forceinline__ void put(float* p, double v) { *p = (float)v; }

template <typename T>
__global__ __launch_bounds__(EW_THREADS) void fill_normal_kernel(T* __restrict__ out, int64_t n, int64_t cols,
                                                                 int64_t ld, uint64_t stream, double scale,
                                                                 double offset, int gu_f) {
  const int64_t i = int64_t(blockIdx.x) * EW_THREADS + threadIdx.x;  // flat index in the dense (public) layout
  if (i >= n) return;
  const uint64_t c = stream + 2ull * (uint64_t)i;
  const uint64_t r1 = mix64(c), r2 = mix64(c + 1);
  const double u1 = ((double)(r1 >> 11) + 1.0) * 0x1p-53;
  const double u2 = (double)(r2 >> 11) * 0x1p-53;
  const double z = sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925286766559 * u2);
  const int64_t col = i % cols;  // gu_f > 0: the tensor is stored in the interleaved gate/up column order
  put(out + (i / cols) * ld + (gu_f > 0 ? gu_interleaved_col(int(col), gu_f) : col), offset + scale * z);
}

// dst <- src with the columns of a [rows, 2f] matrix moved between the public and the interleaved gate/up order
// (8 columns per thread; blocks of 32 columns move as a whole).  The caller's side may begin at any element.
__global__ __launch_bounds__(EW_THREADS) void gu_permute_kernel(const bf16_t* __restrict__ src, int64_t ld_src,
                                                                bf16_t* __restrict__ dst, int64_t ld_dst,
                                                                int64_t total, int f, bool to_interleaved) {
  const int64_t id = int64_t(blockIdx.x) * EW_THREADS + threadIdx.x;
  if (id >= total) return;
  const int cpr = f >> 2;  // 16-byte chunks per row of 2f columns
  const int64_t t = id / cpr;
  const int c = int(id % cpr) * 8, ci = gu_interleaved_col(c, f);
  uint4 v;
  __builtin_memcpy(&v, src + t * ld_src + (to_interleaved ? c : ci), 16);
  __builtin_memcpy(dst + t * ld_dst + (to_interleaved ? ci : c), &v, 16);
}

// ---------------------------------------------------------------- parameters into their places (bf16)
// One launch places up to MAX_SPREAD matrices: dst (row stride ld_dst; columns in the interleaved gate/up order if gu_f > 0)
// and the transposed copy dst_t, from one read of src.  HBM-bound.  128 x 128 tiles, so that every row piece of all three
// matrices is 256 bytes (gate/up: two of 128 in src; a tile is one of the interleaved order, since pieces of lines are dearer to
// write than to read); a tile goes through LDS with the 16-byte chunks of a row XORed by its group of eight rows (the
// transposing reads take one column of 16 groups: 16 different chunks, no bank conflicts).  Rows and columns are
// multiples of 8 wherever dst_t is written.
// Measured (the matrices of a 4096 x 11008 layer, 405 MB in, 810 MB out): 425 us as copies, a column permutation and
// 64 x 64 transposes with 2-byte accesses; 264 us as one pass in tiles of src, 238 in tiles of the interleaved order (5.1 TB/s).  With
// an ffn of 10008, no multiple of 32, 268 and 233, as much as without the interleaving (230).  Small layers are equal within 1 us (of
// eleven shapes one lost: hidden 1464, ffn 2816, two layers 75.5 -> 77.8).
struct SpreadList {
  mls::Spread m[mls::MAX_SPREAD];
  int first[mls::MAX_SPREAD];  // first tile of each matrix
  int n;
};
__host__ __device__ __forceinline__ int spread_cols(const mls::Spread& m) { return m.gu_f > 0 ? 2 * gu_width(m.gu_f) : m.cols; }
__global__ __launch_bounds__(256) void spread_bf16_kernel(SpreadList L) {
  __shared__ uint4 tile[128 * 16];
  int w = 0;
  while (w + 1 < L.n && int(blockIdx.x) >= L.first[w + 1]) w++;
  const mls::Spread& m = L.m[w];
  const bf16_t* src = (const bf16_t*)m.src;
  bf16_t *dst = (bf16_t*)m.dst, *dst_t = (bf16_t*)m.dst_t;
  const int at = int(blockIdx.x) - L.first[w], tx = (spread_cols(m) + 127) / 128;
  const int r0 = at / tx * 128, c0 = at % tx * 128;
  const int ch = threadIdx.x & 15, tr = threadIdx.x >> 4;
  auto exists = [&](int c) { return c < spread_cols(m) && (m.gu_f <= 0 || gu_column_exists(c, m.gu_f)); };
  const int col = c0 + ch * 8, from = m.gu_f > 0 ? gu_public_col(col, m.gu_f) : col;
  const bool some = exists(col);
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const int r = i * 16 + tr;
    if (r0 + r < m.rows && some) {
      const uint4 v = *reinterpret_cast<const uint4*>(src + int64_t(r0 + r) * m.ld_src + from);
      if (dst) *reinterpret_cast<uint4*>(dst + int64_t(r0 + r) * m.ld_dst + col) = v;
      tile[r * 16 + (ch ^ (r >> 3))] = v;
    }
  }
  if (!dst_t) return;
  __syncthreads();
  const uint16_t* t16 = reinterpret_cast<const uint16_t*>(tile);
  const int rg = threadIdx.x & 15;  // rows r0 + 8 rg .. +7
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const int c = i * 16 + (threadIdx.x >> 4), gc = c0 + c;
    if (exists(gc) && r0 + rg * 8 < m.rows) {
      uint32_t e[8];
#pragma unroll
      for (int q = 0; q < 8; q++) e[q] = t16[((rg * 8 + q) * 16 + ((c >> 3) ^ rg)) * 8 + (c & 7)];
      const uint4 v = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
      *reinterpret_cast<uint4*>(dst_t + int64_t(gc) * m.ld_t + r0 + rg * 8) = v;
    }
  }
}

inline int blocks_for(int64_t n) { return int((n + EW_THREADS - 1) / EW_THREADS); }

}  // namespace

namespace mls {

// (below 2048 rows the launch is what either form costs; wider rows are no faster by wavefront: 2 x 4096 rows of 2048 97 and 105 us)
static bool norm_by_wave(int dt, int T, int h) { return dt == DT_BF16 && h <= 1024 && T >= 2048; }

hipError_t rmsnorm_fwd(int dt, const void* x, int64_t ldx, const void* gamma, void* a, int64_t lda, float* r, int T,
                       int h, float eps, hipStream_t st, void* copy, int64_t ldc) {
  if (T == 0) return hipSuccess;
  if (norm_by_wave(dt, T, h)) {
#define FWDW(C)                                                                                                                        \
  hipLaunchKernelGGL((rmsnorm_fwd_wave_kernel<C>), dim3((T + 3) / 4), dim3(EW_THREADS), 0, st, (const bf16_t*)x, ldx, (const bf16_t*)gamma, \
                     (bf16_t*)a, lda, r, T, h, eps, (bf16_t*)copy, ldc)
    if (h <= 512) FWDW(1); else FWDW(2);
#undef FWDW
    return hipGetLastError();
  }
#define FWD(TY, C)                                                                                             \
  hipLaunchKernelGGL((rmsnorm_fwd_kernel<TY, C>), dim3(T), dim3(EW_THREADS), 0, st, (const TY*)x, ldx,             \
                     (const TY*)gamma, (TY*)a, lda, r, h, eps, (TY*)copy, ldc)
  const int mc = h <= 4096 ? 2 : h <= 8192 ? 4 : 8;
  if (dt == DT_BF16) {
    if (mc == 2) FWD(bf16_t, 2); else if (mc == 4) FWD(bf16_t, 4); else FWD(bf16_t, 8);
  } else {
    if (mc == 2) FWD(float, 2); else if (mc == 4) FWD(float, 4); else FWD(float, 8);
  }
#undef FWD
  return hipGetLastError();
}

int rmsnorm_bwd_blocks(int T) { return T < 512 ? (T > 0 ? T : 1) : 512; }

hipError_t rmsnorm_bwd(int dt, const void* da, int64_t ld_da, const void* x, int64_t ldx, const void* gamma,
                       const float* r, const void* dres, int64_t ld_dres, void* dx, int64_t ld_dx, float* dgamma,
                       float* partial, int T, int h, hipStream_t st, bool overwrite, bool acc_partial, bool reduce) {
  if (T == 0) return hipSuccess;
  const int nb = rmsnorm_bwd_blocks(T);
#define BWDW(C)                                                                                                                         \
  hipLaunchKernelGGL((rmsnorm_bwd_wave_kernel<C>), dim3(nb), dim3(EW_THREADS), 0, st, (const bf16_t*)da, ld_da, (const bf16_t*)x, ldx,            \
                     (const bf16_t*)gamma, r, (const bf16_t*)dres, ld_dres, (bf16_t*)dx, ld_dx, partial, T, h, acc_partial)
#define BWD(TY, C)                                                                                               \
  hipLaunchKernelGGL((rmsnorm_bwd_kernel<TY, C>), dim3(nb), dim3(EW_THREADS), 0, st, (const TY*)da, ld_da,            \
                     (const TY*)x, ldx, (const TY*)gamma, r, (const TY*)dres, ld_dres, (TY*)dx, ld_dx, partial, T, h, acc_partial)
  const int mc = h <= 4096 ? 2 : h <= 8192 ? 4 : 8;
  if (norm_by_wave(dt, T, h)) {
    if (h <= 512) BWDW(1); else BWDW(2);
  } else if (dt == DT_BF16) {
    if (mc == 2) BWD(bf16_t, 2); else if (mc == 4) BWD(bf16_t, 4); else BWD(bf16_t, 8);
  } else {
    if (mc == 2) BWD(float, 2); else if (mc == 4) BWD(float, 4); else BWD(float, 8);
  }
#undef BWD
#undef BWDW
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !reduce) return e;
  return rmsnorm_bwd_reduce(rmsnorm_bwd_sums(partial, dgamma, nullptr, nullptr, T, h, overwrite), st);
}

Colsum rmsnorm_bwd_sums(const float* partial0, float* dgamma0, const float* partial1, float* dgamma1, int T, int h, bool overwrite) {
  return {partial0, dgamma0, partial1, dgamma1, rmsnorm_bwd_blocks(T), h, overwrite ? 1 : 0, (h + 15) / 16 * (partial1 ? 2 : 1)};
}
hipError_t rmsnorm_bwd_reduce(const Colsum& cs, hipStream_t st) {
  if (cs.nblocks == 0 || cs.wgs == 0) return hipSuccess;
  hipLaunchKernelGGL(colsum_add_kernel, dim3(cs.wgs), dim3(256), 0, st, cs);
  return hipGetLastError();
}

hipError_t copy_rows(const void* src, int64_t ld_src, int64_t next_src, void* dst, int64_t ld_dst, int64_t next_dst, int64_t bytes,
                     int rows, int n, hipStream_t st) {
  if (rows == 0 || n == 0 || bytes == 0) return hipSuccess;
  if ((bytes | ld_src | ld_dst | next_src | next_dst) & 15) return hipErrorInvalidValue;
  const int64_t cpr = bytes / 16, total = rows * cpr;
  hipLaunchKernelGGL(copy_rows_kernel, dim3(blocks_for(total), n), dim3(EW_THREADS), 0, st, (const char*)src, ld_src, next_src, (char*)dst,
                     ld_dst, next_dst, int(cpr), total);
  return hipGetLastError();
}

// n floats (a multiple of 4, 16-byte aligned) <- 0, as a kernel (safe to record into a HIP graph)
hipError_t fill_zero_f32(float* p, size_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (n % 4 || (uintptr_t(p) & 15)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(unsigned((n / 4 + 255) / 256)), dim3(256), 0, st, reinterpret_cast<float4*>(p), n / 4);
  return hipGetLastError();
}

hipError_t rope_inplace(void* u, const float* cos_tab, const float* sin_tab, int T, int S, int n_heads, int d, int64_t ld, hipStream_t st) {
  const int64_t total = int64_t(T) * n_heads * (d >> 4);
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(rope_kernel, dim3(blocks_for(total)), dim3(EW_THREADS), 0, st, (bf16_t*)u, cos_tab, sin_tab, total, S, n_heads, d, ld);
  return hipGetLastError();
}

hipError_t swiglu_fwd(const void* gu, int64_t ld_gu, void* z, int64_t ld_z, int T, int f, hipStream_t st) {
  const int64_t total = int64_t(T) * (f >> 3);
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(swiglu_fwd_kernel, dim3(blocks_for(total)), dim3(EW_THREADS), 0, st, (const bf16_t*)gu, ld_gu, (bf16_t*)z, ld_z, total, f);
  return hipGetLastError();
}

hipError_t swiglu_bwd(const void* dz, int64_t ld_dz, const void* gu, int64_t ld_gu, void* dgu, int64_t ld_dgu, int T, int f, hipStream_t st,
                      bool interleaved) {
  const int64_t total = int64_t(T) * (f >> 3);
  if (total == 0) return hipSuccess;
  if (interleaved && f % 8) return hipErrorInvalidValue;
  auto kern = interleaved ? swiglu_bwd_kernel<true> : swiglu_bwd_kernel<false>;
  hipLaunchKernelGGL(kern, dim3(blocks_for(total)), dim3(EW_THREADS), 0, st, (const bf16_t*)dz, ld_dz, (const bf16_t*)gu, ld_gu, (bf16_t*)dgu,
                     ld_dgu, total, f);
  return hipGetLastError();
}

hipError_t gu_permute(const void* src, int64_t ld_src, void* dst, int64_t ld_dst, int64_t rows, int f,
                      bool to_interleaved, hipStream_t st) {
  const int64_t total = rows * (f >> 2);
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(gu_permute_kernel, dim3(blocks_for(total)), dim3(EW_THREADS), 0, st, (const bf16_t*)src, ld_src,
                     (bf16_t*)dst, ld_dst, total, f, to_interleaved);
  return hipGetLastError();
}

hipError_t spread_bf16(const Spread* list, int n, hipStream_t st) {
  if (n < 0 || n > MAX_SPREAD) return hipErrorInvalidValue;
  SpreadList L = {};
  int64_t tiles = 0;
  for (int i = 0; i < n; i++) {
    if (list[i].rows <= 0 || list[i].cols <= 0) continue;
    L.m[L.n] = list[i];
    L.first[L.n++] = int(tiles);
    tiles += int64_t((list[i].rows + 127) / 128) * ((spread_cols(list[i]) + 127) / 128);
  }
  if (tiles == 0) return hipSuccess;
  if (tiles > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(spread_bf16_kernel, dim3(unsigned(tiles)), dim3(256), 0, st, L);
  return hipGetLastError();
}

hipError_t fill_normal(int dt, void* out, int64_t rows, int64_t cols, int64_t ld, uint64_t seed, uint32_t tensor,
                       uint32_t layer, double scale, double offset, hipStream_t st, int gu_f) {
  const int64_t n = rows * cols;
  if (n == 0) return hipSuccess;
  auto mixh = [](uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  };
  const uint64_t stream = mixh(mixh(seed) ^ ((uint64_t(tensor) << 32) | layer));
  if (dt == DT_BF16)
    hipLaunchKernelGGL(fill_normal_kernel<bf16_t>, dim3(blocks_for(n)), dim3(EW_THREADS), 0, st, (bf16_t*)out, n, cols,
                       ld, stream, scale, offset, gu_f);
  else
    hipLaunchKernelGGL(fill_normal_kernel<float>, dim3(blocks_for(n)), dim3(EW_THREADS), 0, st, (float*)out, n, cols, ld,
                       stream, scale, offset, gu_f);
  return hipGetLastError();
}

}  // namespace mls
