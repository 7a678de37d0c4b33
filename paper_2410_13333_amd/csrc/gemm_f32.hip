// fp32 GEMM of the all-fp32 validation mode, on v_mfma_f32_32x32x2_f32 (full fp32 products and sums).  Same three modes
// and epilogues as the bf16 kernel.
//
// The shapes of this mode are small, so what bounds a launch is the chain of K / 2 dependent MFMAs of an output tile and
// the number of tiles: the four wavefronts of a workgroup share ONE output tile and take every fourth 32-deep piece of
// the contraction each, and their partial sums meet in a fixed tree through LDS (the same sum order on every run).
// Operands go straight from memory to registers: a lane's MFMA operand is one row (or column) at one k, and since the
// order of the contraction is free as long as both operands agree, the two lane halves take k-values 8g .. 8g+3 and
// 8g+4 .. 8g+7, so that an operand stored along k is read 16 bytes per lane and one stored across it in 128-byte rows.
// The next piece is requested before the MFMAs of the current one.
// Measured (512 tokens, hidden 512: 24 launches of a step, K = 512 .. 2752): 161 us per launch with the scalar-FMA kernel
// this replaced (64x64 tiles through LDS), 21 us with this one.
#include "common.h"
#include "kernels.h"

namespace {

constexpr int KC = 32;  // contraction depth of one piece: whole 128-byte lines of an operand stored along k

// element (row, k) of an operand at base[row * srow + k * sk]; ALONG_K: sk == 1, 16-byte loads (k a multiple of 4 and
// rows 16-byte aligned, which the entry point checks)
template <bool ALONG_K>
__device__ __forceinline__ void load_piece(const float* __restrict__ base, int64_t ld, int row, int k0, int K, int hf,
                                           float (&f)[KC / 2]) {
#pragma unroll
  for (int g = 0; g < KC / 8; g++) {
    const int k = k0 + 8 * g + 4 * hf;
    if (ALONG_K) {  // (K is a multiple of 8 here: groups are whole)
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k0 + 8 * g < K) v = *reinterpret_cast<const float4*>(base + int64_t(row) * ld + k);
      f[4 * g] = v.x; f[4 * g + 1] = v.y; f[4 * g + 2] = v.z; f[4 * g + 3] = v.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; j++) f[4 * g + j] = k + j < K ? base[int64_t(k + j) * ld + row] : 0.f;
    }
  }
}

// One workgroup = one (32 NT) x (32 NT) tile of C.  A(m, k): AK ? A[m*lda + k] : A[k*lda + m]; B(k, n): BK ? B[n*ldb + k]
// : B[k*ldb + n].
template <int NT, bool AK, bool BK>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B, float* C,
                                                       const float* R, int M, int N, int K, int64_t lda, int64_t ldb,
                                                       int64_t ldc, int64_t ldr, int accumulate) {
  __shared__ float part[2][NT * NT * 16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5;
  const int m0 = blockIdx.y * (32 * NT), n0 = blockIdx.x * (32 * NT);
  // rows and columns past the end repeat the last one: their results are not stored
  int ar[NT], bc[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) {
    ar[t] = min(m0 + t * 32 + l32, M - 1);
    bc[t] = min(n0 + t * 32 + l32, N - 1);
  }
  f32x16 acc[NT][NT];
#pragma unroll
  for (int i = 0; i < NT; i++)
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
  float a[2][NT][KC / 2], b[2][NT][KC / 2];
  auto load = [&](int k0, int s) {
#pragma unroll
    for (int t = 0; t < NT; t++) {
      load_piece<AK>(A, lda, ar[t], k0, K, hf, a[s][t]);
      load_piece<BK>(B, ldb, bc[t], k0, K, hf, b[s][t]);
    }
  };
  auto mul = [&](int s) {  // operands swapped: a lane ends up with 4 consecutive columns of one row of C
#pragma unroll
    for (int q = 0; q < KC / 2; q++)
#pragma unroll
      for (int i = 0; i < NT; i++)
#pragma unroll
        for (int j = 0; j < NT; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[s][j][q], a[s][i][q], acc[i][j], 0, 0, 0);
  };
  const int step = 4 * KC;
  int k0 = wave * KC;
  if (k0 < K) load(k0, 0);
  while (k0 < K) {  // two pieces per turn, so that the two register sets need no copies
    if (k0 + step < K) load(k0 + step, 1);
    mul(0);
    k0 += step;
    if (k0 >= K) break;
    if (k0 + step < K) load(k0 + step, 0);
    mul(1);
    k0 += step;
  }
  // wavefronts 2, 3 -> 0, 1; then 1 -> 0
#pragma unroll
  for (int half = 2; half > 0; half >>= 1) {
    if (wave >= half && wave < 2 * half)
#pragma unroll
      for (int i = 0; i < NT; i++)
#pragma unroll
        for (int j = 0; j < NT; j++)
#pragma unroll
          for (int e = 0; e < 16; e++) part[wave - half][(i * NT + j) * 16 + e][lane] = acc[i][j][e];
    __syncthreads();
    if (wave < half)
#pragma unroll
      for (int i = 0; i < NT; i++)
#pragma unroll
        for (int j = 0; j < NT; j++)
#pragma unroll
          for (int e = 0; e < 16; e++) acc[i][j][e] += part[wave][(i * NT + j) * 16 + e][lane];
    __syncthreads();
  }
  if (wave != 0) return;
#pragma unroll
  for (int i = 0; i < NT; i++) {
    const int row = m0 + i * 32 + l32;
    if (row >= M) continue;
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int col = n0 + j * 32 + 8 * g + 4 * hf;  // N is a multiple of 8: groups of four are whole
        if (col >= N) continue;
        float4* c = reinterpret_cast<float4*>(C + int64_t(row) * ldc + col);
        float4 v = make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        if (accumulate) o = *c;
        else if (R) o = *reinterpret_cast<const float4*>(R + int64_t(row) * ldr + col);
        *c = make_float4(v.x + o.x, v.y + o.y, v.z + o.z, v.w + o.w);
      }
  }
}

template <bool AK, bool BK>
void launch_f32(const float* A, const float* B, float* C, const float* R, int M, int N, int K, int64_t lda, int64_t ldb,
                int64_t ldc, int64_t ldr, int acc, hipStream_t st) {
  // 64x64 tiles read half as much per product, 32x32 tiles make four times the workgroups: the big ones once they give
  // every CU two workgroups
  const int64_t big = int64_t((M + 63) / 64) * ((N + 63) / 64);
  if (big >= 512)
    hipLaunchKernelGGL((gemm_f32_kernel<2, AK, BK>), dim3((N + 63) / 64, (M + 63) / 64), dim3(256), 0, st, A, B, C, R, M, N, K,
                       lda, ldb, ldc, ldr, acc);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<1, AK, BK>), dim3((N + 31) / 32, (M + 31) / 32), dim3(256), 0, st, A, B, C, R, M, N, K,
                       lda, ldb, ldc, ldr, acc);
}

}  // namespace

namespace mls {

// M, N and row strides multiples of 8, operands 16-byte aligned (as every entry point checks); K a multiple of 8 in the
// NN and NT forms, any length in the TN form (a weight gradient contracts over the tokens)
hipError_t gemm_f32(int mode, const void* A, const void* B, void* C, const void* R, int M, int N, int K, int64_t lda,
                    int64_t ldb, int64_t ldc, int64_t ldr, hipStream_t st) {
  if (M == 0 || N == 0) return hipSuccess;
  const float *a = (const float*)A, *b = (const float*)B, *r = (const float*)R;
  float* c = (float*)C;
  switch (mode) {
    case GEMM_NN: launch_f32<true, false>(a, b, c, r, M, N, K, lda, ldb, ldc, ldr, 0, st); break;
    case GEMM_NT: launch_f32<true, true>(a, b, c, r, M, N, K, lda, ldb, ldc, ldr, 0, st); break;
    case GEMM_TN: launch_f32<false, false>(a, b, c, r, M, N, K, lda, ldb, ldc, ldr, 1, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace mls
