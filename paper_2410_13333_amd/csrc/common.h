// Shared device helpers of the decoder-stage library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) int i32x2;

#define MLS_LDS __attribute__((address_space(3)))

// ---- loops over compile-time indices
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// ---- raw buffers, requests into LDS, waits: inline asm where the kernels place waits by hand
constexpr uint32_t OOB = 0x80000000u;  // a byte offset beyond every buffer
__device__ __forceinline__ i32x4 make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)p;
  i32x4 r;
  r[0] = (int)(uint32_t)a;
  r[1] = (int)((uint32_t)(a >> 32) & 0xffffu);  // stride 0: raw buffer, byte offsets
  r[2] = (int)bytes;
  r[3] = 0x00020000;
  return r;
}
// 16 bytes per lane from a raw buffer straight into LDS: 64 lanes fill 1 KiB at lds_byte.  soff is a scalar byte
// offset added to the address; it is not part of the range check (voff >= num_records zero-fills).
__device__ __forceinline__ void dma16s(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds_byte) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_byte), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lgkm0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- fragments of 16x16x32 products
// C tile (16 columns x 16 rows, transposed product): lane l ends up with C[row l%16][cols 4*(l/16) .. +3]
__device__ __forceinline__ void mfma16(f32x4& c, const i32x4& bfrag, const i32x4& afrag) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(bfrag), "v"(afrag));
}
template <int OFF>
__device__ __forceinline__ void lds_read16(i32x4& f, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f) : "v"(addr), "n"(OFF) : "memory");
}
// transposing read of a [k][col] tile: two 8-byte reads (k-rows kr and kr+4 of the lane's group of eight); ROW bytes per
// k-row
template <int OFF, int ROW>
__device__ __forceinline__ void lds_read16_tr(i32x4& f, uint32_t addr) {
  i32x2 lo, hi;
  asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
               : "=&v"(lo), "=&v"(hi)
               : "v"(addr), "n"(OFF), "n"(OFF + 4 * ROW)
               : "memory");
  f = i32x4{lo[0], lo[1], hi[0], hi[1]};  // (the two halves are allocated as one register quad: no copies)
}

// ---- 8-element (one 16-byte bf16 chunk / two 16-byte fp32 chunks) loads and stores, values as fp32
__device__ __forceinline__ void load8(const bf16_t* p, float (&v)[8]) {
  uint4 raw = *reinterpret_cast<const uint4*>(p);
  uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; i++) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  bf16x2 t = {(bf16_t)lo, (bf16_t)hi};  // round-to-nearest-even (v_cvt_pk_bf16_f32)
  return __builtin_bit_cast(uint32_t, t);
}
__device__ __forceinline__ void store8(bf16_t* p, const float (&v)[8]) {
  uint4 raw;
  raw.x = pack_bf16x2(v[0], v[1]); raw.y = pack_bf16x2(v[2], v[3]);
  raw.z = pack_bf16x2(v[4], v[5]); raw.w = pack_bf16x2(v[6], v[7]);
  *reinterpret_cast<uint4*>(p) = raw;
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
  reinterpret_cast<float4*>(p)[0] = make_float4(v[0], v[1], v[2], v[3]);
  reinterpret_cast<float4*>(p)[1] = make_float4(v[4], v[5], v[6], v[7]);
}
// ---- 4-element bf16 (8-byte) loads and stores
__device__ __forceinline__ void load4(const bf16_t* p, float (&v)[4]) {
  const uint2 raw = *reinterpret_cast<const uint2*>(p);
  v[0] = __uint_as_float(raw.x << 16);
  v[1] = __uint_as_float(raw.x & 0xffff0000u);
  v[2] = __uint_as_float(raw.y << 16);
  v[3] = __uint_as_float(raw.y & 0xffff0000u);
}
__device__ __forceinline__ void store4(bf16_t* p, const float (&v)[4]) {
  uint2 raw;
  raw.x = pack_bf16x2(v[0], v[1]);
  raw.y = pack_bf16x2(v[2], v[3]);
  *reinterpret_cast<uint2*>(p) = raw;
}
__device__ __forceinline__ float round_bf16(float v) { return (float)(bf16_t)v; }
__device__ __forceinline__ float sigmoidf_(float g) { return 1.f / (1.f + __expf(-g)); }

// ---- gate/up column order.  Public: [gate 0..f) | up 0..f)].  Interleaved (internal, used when the SwiGLU is fused
// into the contractions around it): 32 gate columns, then the 32 up columns of the same indices, and so on, so that a lane of
// the contraction's epilogue holds a gate and its up.  The last group is filled up with zero weights where f % 32 != 0: the
// matrices are then 2 gu_width(f) columns wide.
__host__ __device__ __forceinline__ int gu_width(int f) { return (f + 31) / 32 * 32; }
__host__ __device__ __forceinline__ bool gu_column_exists(int n, int f) { return (n >> 6) * 32 + (n & 31) < f; }
__host__ __device__ __forceinline__ int gu_public_col(int n, int f) { return ((n >> 5) & 1) * f + (n >> 6) * 32 + (n & 31); }
__host__ __device__ __forceinline__ int gu_interleaved_col(int c, int f) {
  const int w = c >= f, r = c - w * f;
  return (r >> 5) * 64 + w * 32 + (r & 31);
}

// ---- contractions shared out over several workgroups: `parts` of them per tile of the result, each over its share of the
// contraction.  All but the last to finish leave their fp32 sums in `sums` (a slot of 256 threads x 16 WTM WTN bytes each) and
// are done; the last one adds them up in the order of the parts, so that the bits do not depend on who came last, and goes on
// to the epilogue.  state: two counters per tile, zero before the launch and after it: who has arrived, whose sums are there.
// No workgroup waits for one that may not have started: the last one waits for stores that are on their way.
// The exchange may cross XCDs, whose L2 caches are not coherent with each other: agent-scope accesses (sc1) on both sides, the
// sums announced when their stores have completed.  (Release and acquire fences of that scope write back and invalidate the
// whole L2 under the other workgroups: 2048 x 4096 x 22016 on 256x256 tiles in two parts 278 us instead of 254.  Announced in
// four pieces, for the reader to start on the first: no faster.)
struct SplitArgs {
  float* sums;
  uint32_t* state;
  int parts;
};
constexpr int CP_AGENT = 16;  // cache policy bit sc1 of the buffer instructions
template <int WTM, int WTN>
__device__ __forceinline__ bool join_parts(const SplitArgs& sp, int tile, int part, f32x4 (&c)[WTM][WTN], uint32_t* word) {
  constexpr int NT = WTM * WTN, SLOT = NT * 256 * 16;
  const int tid = threadIdx.x, parts = sp.parts;
  uint32_t* st = sp.state + 2 * int64_t(tile);
  if (tid == 0) *word = __hip_atomic_fetch_add(st, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const bool last = __builtin_amdgcn_readfirstlane(int(*word)) == parts - 1;
  // (of two parts only one is ever stored)
  auto slot = [&](int p, bool some) {
    const int64_t at = parts == 2 ? tile : int64_t(tile) * parts + p;
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<unsigned char*>(sp.sums) + at * SLOT, 0, some ? SLOT : 0, 0x00020000);
  };
  if (!last) {
    const auto r = slot(part, true);
#pragma unroll
    for (int i = 0; i < NT; i++)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, c[i / WTN][i % WTN]), r, tid * 16, i * 4096, CP_AGENT);
    wait_vmcnt<0>();
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(st + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
  if (tid == 0) {
    while (__hip_atomic_load(st + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != uint32_t(parts - 1)) __builtin_amdgcn_s_sleep(1);
    __hip_atomic_store(st, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(st + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  asm volatile("" ::: "memory");
  auto read = [&](auto r, int i) { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, tid * 16, i * 4096, CP_AGENT)); };
  if (NT >= 32 || parts == 2) {  // two parts: a + b has the bits of b + a
    const auto r = slot(0, true);
    constexpr int B = NT < 16 ? NT : 16;  // read together (64 registers)
#pragma unroll
    for (int b = 0; b < NT; b += B) {
      f32x4 v[B];
#pragma unroll
      for (int i = 0; i < B; i++) v[i] = read(r, b + i);
#pragma unroll
      for (int i = 0; i < B; i++) c[(b + i) / WTN][(b + i) % WTN] += v[i];
      __builtin_amdgcn_sched_barrier(0);
    }
    return true;
  }
  if constexpr (NT < 32) {
    constexpr int AT_ONCE = NT >= 16 ? 1 : 16 / NT;  // parts read together
    f32x4 sum[NT];
#pragma unroll
    for (int i = 0; i < NT; i++) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < parts; p0 += AT_ONCE) {
      f32x4 v[AT_ONCE][NT];
#pragma unroll
      for (int q = 0; q < AT_ONCE; q++) {
        const auto r = slot(p0 + q, p0 + q < parts && p0 + q != part);
#pragma unroll
        for (int i = 0; i < NT; i++) v[q][i] = read(r, i);
      }
#pragma unroll
      for (int q = 0; q < AT_ONCE; q++) {
        const bool own = p0 + q == part;
#pragma unroll
        for (int i = 0; i < NT; i++) sum[i] += own ? c[i / WTN][i % WTN] : v[q][i];
      }
    }
#pragma unroll
    for (int i = 0; i < NT; i++) c[i / WTN][i % WTN] = sum[i];
  }
  return true;
}

// ---- fp32 results of a wavefront's 16x16x32 tiles (lane l holds row l%16 of a block of 16, columns 4 (l/16) .. +3 of a tile):
// C[row0 + 16 i + l%16][..] = c, or += c.  w0: the wavefront's first column, of N; column n lies at col0 + n of C, or, with
// xf > 0, where the interleaved gate/up column col0 + n has its public place.  16 rows of C must span less than 2^31 bytes.
// HBM bounds it (the matrix cores wait meanwhile), so the blocks pass through `ws` (1 KiB * WTN of this wavefront's LDS) and
// memory sees whole lines at once, 64 WTN bytes of a row; and what is added to is read AHEAD blocks before it is needed, since a
// wavefront that is alone on its SIMD has nothing else to hide the latency with.  Rows and columns beyond the ends leave the
// range of the block's descriptor: no branch stands between the loads.  The four weight gradients of a 4096 / 11008 layer over
// 2048 tokens, added: 1066 us with each load used at once and 64 bytes of a row per access, 923 read ahead, 884 in rows
// (stored: 766, 733, 705).
template <int WTM, int WTN>
__device__ __forceinline__ void f32_results(float* C, int64_t ldc, int row0, int M, int w0, int N, int col0, int xf, bool add,
                                            const f32x4 (&c)[WTM][WTN], int lane, unsigned char* ws) {
  constexpr int CH = 4 * WTN, RPI = 64 / CH, NQ = WTN;  // 16-byte chunks per row, rows per access, accesses per block
  const int l16 = lane & 15, g4 = lane >> 4, chk = lane % CH, r0 = lane / CH;
  const int n = w0 + chk * 4;
  const int64_t at = xf > 0 ? gu_public_col(col0 + n, xf) : col0 + n;
  const bool some = n < N && (xf <= 0 || gu_column_exists(col0 + n, xf));
  int off[NQ];
#pragma unroll
  for (int q = 0; q < NQ; q++) off[q] = some ? int(((q * RPI + r0) * ldc + at) * 4) : int(OOB);
  auto block = [&](int i) {
    const int r = row0 + 16 * i, rows = r >= M ? 0 : M - r < 16 ? M - r : 16;
    return __builtin_amdgcn_make_buffer_rsrc(C + (rows > 0 ? int64_t(r) * ldc : 0), 0, int(rows * ldc * 4), 0x00020000);
  };
  constexpr int AHEAD = WTM < 32 / WTN ? WTM : 32 / WTN;  // 128 registers
  f32x4 t[WTM][NQ];
  auto get = [&](int i) {
#pragma unroll
    for (int q = 0; q < NQ; q++) t[i][q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(block(i), off[q], 0, 0));
  };
  if (add) {
#pragma unroll
    for (int i = 0; i < AHEAD; i++) get(i);
  }
#pragma unroll
  for (int i = 0; i < WTM; i++) {
#pragma unroll
    for (int j = 0; j < WTN; j++) *reinterpret_cast<f32x4*>(ws + l16 * (CH * 16) + (((j * 4 + g4) ^ (l16 & (CH - 1))) << 4)) = c[i][j];
    wave_lds_sync();
    f32x4 v[NQ];
#pragma unroll
    for (int q = 0; q < NQ; q++) {
      const int r = q * RPI + r0;
      v[q] = *reinterpret_cast<const f32x4*>(ws + r * (CH * 16) + ((chk ^ (r & (CH - 1))) << 4));
    }
    wave_lds_sync();
    if (add) {
#pragma unroll
      for (int q = 0; q < NQ; q++) v[q] = t[i][q] + v[q];
      if (i + AHEAD < WTM) get(i + AHEAD);
    }
#pragma unroll
    for (int q = 0; q < NQ; q++) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[q]), block(i), off[q], 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ---- out[c] (+)= sum_b partial[b][c] for one or two pairs (mls::Colsum): workgroup `w` of 256 threads takes 16 columns, 16 row groups
// per column, in a fixed summation order.  What bounds it is the latency of a thread's up to 32 loads: eight are in flight at
// a time, and the two gains of a layer share a launch (two launches that loaded one by one: 2 x 11 us at hidden 1024, 2 x 6.6 at
// 256; then 4.7 and 2.7), or go along with the layer's weight gradients.
constexpr int COLSUM_LDS = 16 * 17;  // floats
template <class Colsum>
__device__ __forceinline__ void colsum_block(const Colsum& cs, int w, float* red) {
  const int per = (cs.h + 15) / 16;
  const bool second = w >= per;
  const float* partial = second ? cs.partial1 : cs.partial0;
  float* out = second ? cs.out1 : cs.out0;
  const int cl = threadIdx.x & 15, grp = threadIdx.x >> 4, h = cs.h;
  const int c = (second ? w - per : w) * 16 + cl;
  float s = 0.f;
  if (c < h) {
    int b = grp;
    for (; b + 112 < cs.nblocks; b += 128) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; i++) v[i] = partial[int64_t(b + 16 * i) * h + c];
#pragma unroll
      for (int i = 0; i < 8; i++) s += v[i];
    }
    for (; b < cs.nblocks; b += 16) s += partial[int64_t(b) * h + c];
  }
  red[grp * 17 + cl] = s;
  __syncthreads();
  if (grp == 0 && c < h) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 16; g++) t += red[g * 17 + cl];
    out[c] = cs.overwrite ? t : out[c] + t;
  }
}

__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ void from_f32(bf16_t& d, float v) { d = (bf16_t)v; }
__device__ __forceinline__ void from_f32(float& d, float v) { d = v; }

// ---- reductions: 64-lane wavefront, then up to 16 wavefronts through LDS
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// sum over the whole workgroup; `red` is an LDS array of >= blockDim.x/64 floats; all threads get the result
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();  // protects `red` against the previous use
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; i++) t += red[i];
  return t;
}
