// HBM-streaming workload kernels as logical-block bodies: SAXPY, sum reduction, GEMV,
// row softmax, row LayerNorm.  All are bandwidth-bound: 16-byte coalesced loads, one
// 64-lane wave per row for the row-wise kernels, cross-lane reductions without LDS
// where a wave owns the whole row.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/tally.h"

namespace tally {

constexpr int kThreads = 256;
constexpr int kWave = 64;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;

// Butterflies over a wave.  A shuffle through LDS costs about a hundred cycles a step, six in a
// row for every sum or maximum of a row; here the halves and the 16-lane rows are exchanged by
// the lane swaps and what lies within a row by DPP operands, a few cycles a step.  The partners
// are those of an xor by 32, 16, 8, 4, 2 and 1 in this order (a rotation by 4 pairs the same
// values as an xor by 4 once both lanes of an xor by 8 hold the same), so the sums are the same
// bits.
template <int CTRL>
__device__ __forceinline__ float lane_dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
struct AddOp { static __device__ __forceinline__ float of(float a, float b) { return a + b; } };
struct MaxOp { static __device__ __forceinline__ float of(float a, float b) { return fmaxf(a, b); } };
// over each row of 16 lanes
template <class F>
__device__ __forceinline__ float row16_all(float v) {
  v = F::of(v, lane_dpp<0x128>(v));                        // row_ror:8
  v = F::of(v, lane_dpp<0x124>(v));                        // row_ror:4
  v = F::of(v, lane_dpp<0x4e>(v));                         // quad_perm:[2,3,0,1]
  return F::of(v, lane_dpp<0xb1>(v));                      // quad_perm:[1,0,3,2]
}
// over lanes l, l xor 16, l xor 32 and l xor 48.  (Assembly: the compiler reads the swap
// builtins' two results from one register.  A swap needs two wait states after the vector
// instruction that wrote its operands.)
template <class F>
__device__ __forceinline__ float across_rows(float v) {
  float w = v;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(v), "+v"(w));
  v = F::of(v, w);
  w = v;
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(v), "+v"(w));
  return F::of(v, w);
}
__device__ __forceinline__ float wave_sum(float v) { return row16_all<AddOp>(across_rows<AddOp>(v)); }
__device__ __forceinline__ float wave_max(float v) { return row16_all<MaxOp>(across_rows<MaxOp>(v)); }

// Best-effort forms stream their data with non-temporal accesses (NT): what a best-effort
// kernel reads once and writes once would otherwise push the high-priority job's weights
// and caches out of the L2s and the 256 MB Infinity Cache between two of its requests
// (measured: a decode step beside a streaming softmax took 65 us instead of 41 on the
// device with ordinary accesses, 36 us with non-temporal ones).  The original form of a
// kernel keeps ordinary accesses.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_nt __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ float4 ld4(const float *p) {
  if constexpr (NT) {
    const f32x4_nt v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_nt *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
  } else {
    return *reinterpret_cast<const float4 *>(p);
  }
}
template <bool NT>
__device__ __forceinline__ void st4(float *p, float4 v) {
  if constexpr (NT) {
    const f32x4_nt w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<f32x4_nt *>(p));
  } else {
    *reinterpret_cast<float4 *>(p) = v;
  }
}
template <bool NT>
__device__ __forceinline__ float ld1(const float *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT>
__device__ __forceinline__ void st1(float *p, float v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

#ifdef __HIP_DEVICE_COMPILE__   // (buffer resources have no type in the host compiler's pass)
// A buffer of `bytes` bytes: 16-byte reads past its end give zeros.
typedef __amdgpu_buffer_rsrc_t buf_t;
__device__ __forceinline__ buf_t make_buf(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00027000);
}
__device__ __forceinline__ uint4 buf_ld16(buf_t b, uint32_t byte, uint32_t scalar_byte) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(b, byte, scalar_byte, 0));
}
template <bool NT>
__device__ __forceinline__ float4 buf_ld4(buf_t b, uint32_t byte) {   // (aux bit 1: non-temporal)
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(b, byte, 0, NT ? 2 : 0));
}
#endif

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;  // NaN
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// ---- SAXPY: thread t of block b handles element 256 b + t ----------------------------
struct SaxpyBody {
  using Args = tally_saxpy_args;
  static constexpr bool TEAMS = true;
  static uint64_t block_bytes(const Args &) { return 12 * kThreads; }
  // (us and us of drain with the counter alone / in teams, 2^26: 512 x 8 405 13.1 / 174 7.7, 512 x 24 168 11.8 /
  // 144 10.7, 512 x 32 147 11.8 / 144 12.2; 384 x 16 227 10.4 / 166 8.8; 256 x 8 402 8.4 / 274 7.0, 256 x 16 233 7.9 /
  // 214 8.1.  Blocks beside eights are taken one by one, longer than 256 workers queue: 256 x 12 323 7.5 / 347 9.1)
  static uint32_t team_bytes(uint32_t workers, uint32_t chunk) {
    return workers >= 512 ? 72 << 10 : workers >= 384 || chunk <= 4 || chunk % 8 == 0 ? 48 << 10 : 0;
  }
  static constexpr int THREADS = kThreads;
  static constexpr int MIN_WAVES = 4;
  static constexpr unsigned DYN_LDS = 0;
  static constexpr bool YIELDS = false;
  static constexpr bool END_BARRIER = false;
  static constexpr bool RANGE = true;
  static constexpr bool TOGETHER = true;                  // run_range takes eight blocks at a time
  template <bool NT>
  static __device__ __forceinline__ void run_t(const Args &a, uint32_t bx) {
    uint32_t i = bx * kThreads + threadIdx.x;
    if (i < a.n) st1<NT>(a.y + i, __builtin_fmaf(a.a, ld1<NT>(a.x + i), ld1<NT>(a.y + i)));
  }
  static __device__ __forceinline__ void run(const Args &a, uint32_t bx, uint32_t, uint32_t) { run_t<false>(a, bx); }
  static __device__ __forceinline__ void run_be(const Args &a, uint32_t bx, uint32_t, uint32_t) { run_t<true>(a, bx); }
  // Logical blocks [first, last) of the (one-dimensional) grid in one go, for a worker that
  // fetched several consecutive task indices: the same elements get the same arithmetic as
  // block by block, but the loads of eight blocks are in flight together instead of one
  // block's loads waiting for the previous block's store.
  static __device__ __forceinline__ void run_range(const Args &a, uint32_t first, uint32_t last) {
    // (counted from the first element: the one after 2^32 - 1 of them has no 32-bit index)
    const uint32_t base = first * kThreads, want = (last - first) * kThreads;
    const float *__restrict__ x = a.x + base;
    float *__restrict__ y = a.y + base;
    const uint32_t end = a.n - base < want ? a.n - base : want;
    uint32_t i = threadIdx.x;
    for (; i + 7 * kThreads < end; i += 8 * kThreads) {
      float xv[8], yv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { xv[u] = ld1<true>(x + i + u * kThreads); yv[u] = ld1<true>(y + i + u * kThreads); }
#pragma unroll
      for (int u = 0; u < 8; ++u) st1<true>(y + i + u * kThreads, __builtin_fmaf(a.a, xv[u], yv[u]));
    }
    for (; i < end; i += kThreads) st1<true>(y + i, __builtin_fmaf(a.a, ld1<true>(x + i), ld1<true>(y + i)));
  }
};

// ---- sum reduction: block b -> partial[b] over 4096 consecutive elements --------------
struct ReduceSumBody {
  using Args = tally_reduce_sum_args;
  static constexpr bool TEAMS = true;
  static uint64_t block_bytes(const Args &) { return 4 * PER_BLOCK; }
  // (us and us of drain with the counter alone / in teams, 2^28: 512 x 4 249 12.9 / 169 10.1, 512 x 5 220 12.4 / 172
  // 11.9, 512 x 6 203 12.4 / 172 13.1, 512 x 8 186 13.8 / 174 16.1, 1024 x 2 427 20.6 / 171 10.6; 448 x 5 221 11.4 both;
  // 256 x 4 260 8.4 / 216 8.1.  Blocks beside fours are taken one by one: 256 x 3 309 7.3 / 326 8.5, 384 x 3 302
  // 10.1 / 243 9.4)
  static uint32_t team_bytes(uint32_t workers, uint32_t chunk) {
    return workers >= 512 ? 80 << 10 : workers >= 384 || chunk != 3 ? 64 << 10 : 0;
  }
  static constexpr int THREADS = kThreads;
  static constexpr int MIN_WAVES = 4;
  static constexpr unsigned DYN_LDS = 0;
  static constexpr bool YIELDS = false;
  static constexpr bool RANGE = true;
  static constexpr bool TOGETHER = true;                  // run_range takes four blocks at a time
  static constexpr bool END_BARRIER = false;
  static constexpr uint32_t PER_BLOCK = 4096;
  static __device__ __forceinline__ void run(const Args &a, uint32_t bx, uint32_t, uint32_t) { run_t<false>(a, bx); }
  static __device__ __forceinline__ void run_be(const Args &a, uint32_t bx, uint32_t, uint32_t) { run_t<true>(a, bx); }
  template <bool NT>
  static __device__ __forceinline__ void run_t(const Args &a, uint32_t bx) {
    // two sets of wave partials, alternating with the block index: a worker that runs
    // consecutive blocks back to back then needs no barrier between them (the barrier
    // below already keeps any wave at most one block ahead of the reader)
    __shared__ float s_part2[2][kThreads / kWave];
    float *s_part = s_part2[bx & 1];
    const uint64_t base = (uint64_t)bx * PER_BLOCK;
    float s = 0.f;
    if (base + PER_BLOCK <= a.n) {
      const float *p = a.x + base + 4 * threadIdx.x;
      float4 v0 = ld4<NT>(p), v1 = ld4<NT>(p + 1024), v2 = ld4<NT>(p + 2048), v3 = ld4<NT>(p + 3072);
      s = ((v0.x + v0.y) + (v0.z + v0.w)) + ((v1.x + v1.y) + (v1.z + v1.w)) +
          (((v2.x + v2.y) + (v2.z + v2.w)) + ((v3.x + v3.y) + (v3.z + v3.w)));
    } else {
      for (uint64_t i = base + threadIdx.x; i < a.n; i += kThreads) s += a.x[i];
    }
    s = wave_sum(s);
    if ((threadIdx.x & (kWave - 1)) == 0) s_part[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) a.partial[bx] = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
  }
  // Consecutive blocks [first, last) for a worker that fetched several task indices: four
  // blocks at a time, their 64 KB requested together before any of them is reduced, and one
  // barrier for the four (a persistent worker has far fewer blocks in flight per compute unit
  // than the hardware keeps when it dispatches the original grid, so it has to ask for more
  // per block-time to keep the memory system as busy).  Per block the same sums in the same
  // order as run().
  static __device__ __forceinline__ void run_range(const Args &a, uint32_t first, uint32_t last) {
    __shared__ float s_quad[2][4][kThreads / kWave];
    const uint32_t t = threadIdx.x;
    uint32_t b = first;
    for (uint32_t it = 0; b + 4 <= last && ((uint64_t)b + 4) * PER_BLOCK <= a.n; b += 4, ++it) {
      float4 v[4][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float *p = a.x + (uint64_t)(b + q) * PER_BLOCK + 4 * t;
        v[q][0] = ld4<true>(p); v[q][1] = ld4<true>(p + 1024); v[q][2] = ld4<true>(p + 2048); v[q][3] = ld4<true>(p + 3072);
      }
      float (*part)[kThreads / kWave] = s_quad[it & 1];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float s = ((v[q][0].x + v[q][0].y) + (v[q][0].z + v[q][0].w)) +
                  ((v[q][1].x + v[q][1].y) + (v[q][1].z + v[q][1].w)) +
                  (((v[q][2].x + v[q][2].y) + (v[q][2].z + v[q][2].w)) +
                   ((v[q][3].x + v[q][3].y) + (v[q][3].z + v[q][3].w)));
        s = wave_sum(s);
        if ((t & (kWave - 1)) == 0) part[q][t / kWave] = s;
      }
      __syncthreads();   // (the other buffer is free again: its reader is past this barrier)
      if (t < 4) a.partial[b + t] = (part[t][0] + part[t][1]) + (part[t][2] + part[t][3]);
    }
    for (; b < last; ++b) run_t<true>(a, b);
  }
};

struct ReduceFinalBody {
  using Args = tally_reduce_final_args;
  static constexpr bool TEAMS = false;
  static uint64_t block_bytes(const Args &a) { return 4 * (uint64_t)a.count; }
  static uint32_t team_bytes(uint32_t, uint32_t) { return 0; }   // one block
  static constexpr int THREADS = kThreads;
  static constexpr int MIN_WAVES = 8;   // <= 64 registers: as many may be resident as ever
  static constexpr unsigned DYN_LDS = 0;
  static constexpr bool YIELDS = false;
  static constexpr bool RANGE = false;
  static constexpr bool END_BARRIER = true;   // s_d is reused by the next block
  static __device__ __forceinline__ void run_be(const Args &a, uint32_t x, uint32_t y, uint32_t z) { run(a, x, y, z); }
  // The grid is ONE block, so what bounds it is how many bytes one compute unit keeps on their
  // way: a thread asks for eight 16-byte pieces before it uses the first (32 KB per trip).
  // With one 4-byte element per thread and trip, 65536 partials were 256 memory latencies in a
  // row: 64 us against 6 now (1 GiB sum with its final pass: 256 -> 198 us).
  static __device__ __forceinline__ void run(const Args &a, uint32_t, uint32_t, uint32_t) {
#ifdef __HIP_DEVICE_COMPILE__
    __shared__ double s_d[kThreads / kWave];
    constexpr uint32_t U = 8, TRIP = U * kThreads;         // vectors per trip
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));   // (a worker has no registers to keep the addresses in)
    // partial[] need not be 16-byte aligned: up to three elements before the first whole vector
    const uint32_t mis = (uint32_t)(reinterpret_cast<uintptr_t>(a.partial) >> 2) & 3u;
    const uint32_t lead = mis ? 4u - mis : 0u, head = lead < a.count ? lead : a.count;
    const float *v = a.partial + head;
    const uint32_t nv = (a.count - head) / 4, tail = head + nv * 4;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (uint32_t i = 0; i < nv; i += TRIP, v += 4 * TRIP) {   // (nv < 2^30: no wrap)
      const buf_t b = make_buf(v, (nv - i < TRIP ? nv - i : TRIP) * 16);
      float4 f[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) f[u] = buf_ld4<false>(b, (u * kThreads + t) * 16);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        s0 += (double)f[u].x; s1 += (double)f[u].y; s2 += (double)f[u].z; s3 += (double)f[u].w;
      }
    }
    if (t < head) s0 += (double)a.partial[t];
    if (t < a.count - tail) s1 += (double)a.partial[tail + t];
    double s = (s0 + s1) + (s2 + s3);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
    if ((t & (kWave - 1)) == 0) s_d[t / kWave] = s;
    __syncthreads();
    if (t == 0) *a.total = (s_d[0] + s_d[1]) + (s_d[2] + s_d[3]);
#endif
  }
};

// ---- GEMV: one wave per output row, 16-byte loads along K -----------------------------
struct GemvBody {
  using Args = tally_gemv_bf16_args;
  static constexpr bool TEAMS = true;
  static uint64_t block_bytes(const Args &a) { return 8 * (uint64_t)a.k; }
  // (us and us of drain with the counter alone / in teams: 16384 x 4096, 512 x 1 69 12.4 / 37 7.5; 50000 x 1000,
  // 256 x 1 162 8.5 / 102 6.8, 512 x 4 57 11.4 / 43 8.9)
  static uint32_t team_bytes(uint32_t workers, uint32_t) { return workers >= 512 ? 32 << 10 : 8 << 10; }
  static constexpr int THREADS = kThreads;
  static constexpr int MIN_WAVES = 8;   // <= 64 registers: two waves fit beside a GEMM tile
  static constexpr unsigned DYN_LDS = 0;
  static constexpr bool YIELDS = false;
  static constexpr bool RANGE = false;
  static constexpr bool END_BARRIER = false;
  // 8 bf16 products per 16-byte pair with four packed dot-product instructions (fp32
  // accumulate): a sixth of the vector-ALU work of unpack + fma, which matters because
  // a high-priority GEMV may share its SIMDs with a best-effort GEMM's MFMA stream
  static __device__ __forceinline__ float dot8(uint4 w, uint4 x, float s) {
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.x),
                                        __builtin_bit_cast(bf16x2_t, x.x), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.y),
                                        __builtin_bit_cast(bf16x2_t, x.y), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.z),
                                        __builtin_bit_cast(bf16x2_t, x.z), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.w),
                                        __builtin_bit_cast(bf16x2_t, x.w), s, false);
    return s;
  }
  // (the best-effort forms keep four loads in flight: their loop has no registers to spare)
  static __device__ __forceinline__ void run_be(const Args &a, uint32_t x, uint32_t y, uint32_t z) { run_t<false>(a, x, y, z); }
  static __device__ __forceinline__ void run(const Args &a, uint32_t x, uint32_t y, uint32_t z) { run_t<true>(a, x, y, z); }
  // `left` vectors of a row, N to a lane, from buffers that end with the row: a lane past it gets zeros, which
  // add nothing
  template <int N, bool DEEP>
  static __device__ __forceinline__ void rest(const uint4 *w, const uint4 *x, uint32_t left, uint32_t lane, float &acc0,
                                              float &acc1, float &acc2, float &acc3) {
#ifdef __HIP_DEVICE_COMPILE__
    const buf_t rw = make_buf(w, left * 16), rx = make_buf(x, left * 16);
    uint4 wv[N];
#pragma unroll
    for (int j = 0; j < N; ++j) wv[j] = buf_ld16(rw, lane * 16, j * kWave * 16);
    uint4 xv[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (DEEP || j == 0) {
#pragma unroll
        for (int i = j; i < (DEEP ? j + 1 : N); ++i) xv[i] = buf_ld16(rx, lane * 16, i * kWave * 16);
        // (in a worker the compiler would wait for each of x's loads before the next)
        if constexpr (!DEEP) __builtin_amdgcn_sched_barrier(0);
      }
      float &acc = j % 4 == 0 ? acc0 : j % 4 == 1 ? acc1 : j % 4 == 2 ? acc2 : acc3;
      acc = dot8(wv[j], xv[j], acc);
      if (j == 3) __builtin_amdgcn_sched_barrier(0);       // (x's loads by fours, for the registers)
    }
#endif
  }
  template <bool DEEP>
  static __device__ __forceinline__ void run_t(const Args &a, uint32_t bx, uint32_t, uint32_t) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t row = bx * 4 + threadIdx.x / kWave;
    if (row >= a.n) return;  // wave-uniform; the body holds no barrier
    const uint32_t nvec = a.k / 8;
    const uint4 *w = reinterpret_cast<const uint4 *>(a.W + (uint64_t)row * a.k);
    const uint4 *x = reinterpret_cast<const uint4 *>(a.x);
    float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;   // vector j of a lane goes to accumulator j mod 4
    uint32_t first = 0;                                    // of the batch
    // Batches of eight 16-byte loads of the row per lane (8 KB per wave; a 4096-wide row is
    // one such batch).  Beside the paused tiles of a best-effort GEMM only two of these
    // waves fit on a SIMD, and with four loads each the eight waves of a compute unit had
    // 32 KB on their way where the HBM's latency times the unit's share of its bandwidth
    // asks for ~45 KB: the decode-like request ran at 4.3 TB/s co-located against 5.6 alone.
    // The operand x comes from the caches.  Loads return in order, so each of the first four of the row is followed by
    // x's, and the last four take registers that the first products leave free, within the 64 that let two waves
    // fit (4096 x 4096 from memory 7.05 us; all eight of the row first 7.30, in the compiler's order 7.20).
    for (; DEEP && first + 8 * kWave <= nvec; first += 8 * kWave) {
      const uint32_t v = first + lane;
      const uint4 w0 = w[v], x0 = x[v], w1 = w[v + kWave], x1 = x[v + kWave];
      const uint4 w2 = w[v + 2 * kWave], x2 = x[v + 2 * kWave], w3 = w[v + 3 * kWave], x3 = x[v + 3 * kWave];
      const uint4 x4 = x[v + 4 * kWave], x5 = x[v + 5 * kWave];
      __builtin_amdgcn_sched_barrier(0);
      acc0 = dot8(w0, x0, acc0);
      acc1 = dot8(w1, x1, acc1);
      acc2 = dot8(w2, x2, acc2);
      const uint4 x6 = x[v + 6 * kWave], x7 = x[v + 7 * kWave];
      const uint4 w4 = w[v + 4 * kWave], w5 = w[v + 5 * kWave], w6 = w[v + 6 * kWave], w7 = w[v + 7 * kWave];
      __builtin_amdgcn_sched_barrier(0);
      acc3 = dot8(w3, x3, acc3);
      acc0 = dot8(w4, x4, acc0);
      acc1 = dot8(w5, x5, acc1);
      acc2 = dot8(w6, x6, acc2);
      acc3 = dot8(w7, x7, acc3);
    }
    for (; !DEEP && first + 4 * kWave <= nvec; first += 4 * kWave) {
      const uint32_t v = first + lane;
      uint4 w0 = w[v], w1 = w[v + kWave], w2 = w[v + 2 * kWave], w3 = w[v + 3 * kWave];
      acc0 = dot8(w0, x[v], acc0);
      acc1 = dot8(w1, x[v + kWave], acc1);
      acc2 = dot8(w2, x[v + 2 * kWave], acc2);
      acc3 = dot8(w3, x[v + 3 * kWave], acc3);
    }
    // What is left of the row is one batch more: taken four vectors and then one by one it was up to four
    // memory latencies in a row (us so / now: 700 x 16000 5.7 / 4.4, 3000 x 3592 4.7 / 3.3, 8425 x 1616 6.1 / 4.1),
    // and asking for eight where there are five costs as much as eight (7771 x 2224 6.1 / 5.0, from memory 9.2 / 7.3).
    // The row is made known to be the same in a wave, so that the buffers' descriptors are in scalar registers.
    if (const uint32_t left = nvec - first) {
      const uint4 *e = reinterpret_cast<const uint4 *>(a.W + (uint64_t)__builtin_amdgcn_readfirstlane(row) * a.k) + first;
      switch ((left + kWave - 1) / kWave) {
        case 1: rest<1, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3); break;
        case 2: rest<2, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3); break;
        case 3: rest<3, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3); break;
        case 4: rest<4, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3); break;
        case 5: if constexpr (DEEP) rest<5, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3); break;
        case 6: if constexpr (DEEP) rest<6, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3); break;
        case 7: if constexpr (DEEP) rest<7, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3); break;
        default: if constexpr (DEEP) rest<8, DEEP>(e, x + first, left, lane, acc0, acc1, acc2, acc3);
      }
    }
    float s = wave_sum((acc0 + acc1) + (acc2 + acc3));
    if (lane == 0) a.y[row] = f32_to_bf16(s);
  }
};

// ---- row-wise kernels: softmax and LayerNorm over fp32 rows ---------------------------
// A row is held in registers by a GROUP of lanes, NV float4 each: a wave for rows of up to
// 4096 columns, the whole workgroup for wider ones (a wave would need 128 registers for the
// row alone, and walking such rows three times out of the caches took 393 us for 9001 x 8192,
// 590 MB).  What bounds these kernels is bytes on their way: a persistent worker is often the
// only workgroup of its compute unit, so it keeps DEPTH rows per group in flight: the loads of
// a row are issued as soon as the registers of the row DEPTH before it have been stored.
//
// Rows are addressed as buffers of exactly their own length: a lane past the end reads zeros
// and writes nothing, and a row past the last one is a buffer of length zero.  So there is no
// branch around a load, and with it none of the waits for everything outstanding that the
// compiler places where two paths meet.  A single row per group (every form but a fetch of
// several blocks) has nothing to wait for but itself and takes ordinary loads under a mask,
// which stream up to 8 % faster than buffer loads; so do the stores.
//
// Softmax 9001 x 8192 as 256 workers x 4: 415 -> 150 us (3.9 TB/s), original form 208 -> 116
// (5.1, what a copy reaches); 200000 x 300 as 256 x 4: 308 -> 180 us, bound by the task
// counter (12500 fetches at 11 ns) and a round trip per fetch.
#ifdef __HIP_DEVICE_COMPILE__
__device__ __forceinline__ buf_t row_buf(const float *base, uint64_t row, uint32_t cols, bool exists) {
  return make_buf(base + row * cols, exists ? cols * 4 : 0u);
}
#endif

// Is float4 i of a lane within the row?  The first half of the NV always are: a row that needed no
// more would be held in half as many.  (Softmax 1557 x 1324 4.14 us without this, 4.00 with it.)
template <uint32_t LANES, int NV>
__device__ __forceinline__ bool row_has(uint32_t cols, int i, uint32_t lane) {
  return i < NV / 2 || (i * LANES + lane) * 4 < cols;
}

// A group of LANES threads; `part` is LDS that the waves of a workgroup-wide group share sums
// and maxima through.  Each use is followed by a barrier, and between two uses of one array
// lies the barrier of the other: neither is overwritten while a wave still reads it.
template <uint32_t LANES>
struct RowGroup {
  static constexpr bool WAVE = LANES == (uint32_t)kWave;
  static constexpr uint32_t STEP = WAVE ? kThreads / kWave : 1;   // groups in a workgroup
  static __device__ __forceinline__ void share(float *part, float v) {
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = v;
    __syncthreads();
  }
  static __device__ __forceinline__ float sum(float v, float *part) {
    v = wave_sum(v);
    if constexpr (WAVE) return v;
    share(part, v);
    return (part[0] + part[1]) + (part[2] + part[3]);
  }
  static __device__ __forceinline__ float max(float v, float *part) {
    v = wave_max(v);
    if constexpr (WAVE) return v;
    share(part, v);
    return fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
  }
};

// Op::row(args, row, lane, v) on the `count` rows from r0: group g takes r0 + g, r0 + g + STEP, ...
// (Counted from r0: the row after a matrix of nearly 2^32 rows has no 32-bit number.)
template <class Op, uint32_t LANES, int NV, int DEPTH, bool NT, bool ONE = false>
__device__ __forceinline__ void rows_walk(const typename Op::Args &a, uint32_t r0, uint32_t count) {
#ifdef __HIP_DEVICE_COMPILE__
  typedef RowGroup<LANES> G;
  __shared__ float s_part[2][kThreads / kWave];
  uint32_t lane = threadIdx.x & (LANES - 1);
  uint32_t r = G::WAVE ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : 0u;
  float4 v[DEPTH][NV];
  auto load = [&](uint32_t row, float4 (&x)[NV]) {
    if constexpr (ONE) {
      const float *p = a.x + (uint64_t)(r0 + row) * a.cols;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row_has<LANES, NV>(a.cols, i, lane)) x[i] = ld4<NT>(p + (i * LANES + lane) * 4);
      }
    } else {
      const buf_t b = row_buf(a.x, r0 + row, a.cols, row < count);
#pragma unroll
      for (int i = 0; i < NV; ++i) x[i] = buf_ld4<NT>(b, (i * LANES + lane) * 16);
    }
  };
  // (opaque, and again for each row: a worker would otherwise keep every address that derives
  // from it, and LayerNorm's gamma and beta, in registers across its whole loop)
  asm volatile("" : "+v"(lane));
  if constexpr (ONE) {                                     // a logical block has one row per group
    if (r >= count) return;
    load(r, v[0]);
    Op::template row<G, LANES, NV, NT, true>(a, r0 + r, lane, v[0], s_part[0], s_part[1]);
    return;
  }
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(r + d * G::STEP, v[d]);
  for (;; r += DEPTH * G::STEP) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const uint32_t row = r + d * G::STEP;
      if (row >= count) return;                            // uniform over the group
      asm volatile("" : "+v"(lane));
      Op::template row<G, LANES, NV, NT, false>(a, r0 + row, lane, v[d], s_part[0], s_part[1]);
      if (DEPTH > 1) load(row + DEPTH * G::STEP, v[d]);
    }
    if constexpr (DEPTH == 1) {
      if (r + G::STEP >= count) return;
      load(r + G::STEP, v[0]);
    }
  }
#endif
}

// `v` where the lane is within the row, else `other`: a select, never a branch around what
// computes v (which would split the loads' block and wait for all of them)
__device__ __forceinline__ float row_pick(bool in, float v, float other) {
  asm("" : "+v"(v));
  return in ? v : other;
}

struct SoftmaxOp {
  using Args = tally_softmax_f32_args;
  // (512 workers, us and us of drain with the counter alone / in teams: 60000 x 2048 x 1 block 210 12.2 / 167 11.6,
  // 200000 x 512 x 4 181 11.9 / 147 11.8; 300000 x 200 x 8 139 11.1 / 139 10.6, x 10 123 10.6 / 133 11.9)
  static uint32_t team_bytes(uint32_t chunk) { return chunk <= 8 ? 64 << 10 : 0; }
  template <class G, uint32_t LANES, int NV, bool NT, bool ONE>
  static __device__ __forceinline__ void row(const Args &a, uint32_t r, uint32_t lane, float4 (&v)[NV],
                                             float *part0, float *part1) {
#ifdef __HIP_DEVICE_COMPILE__
    auto in = [&](int i) { return row_has<LANES, NV>(a.cols, i, lane); };
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      m = fmaxf(m, row_pick(in(i), fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)), -INFINITY));
    m = G::max(m, part0);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i].x = __expf(v[i].x - m); v[i].y = __expf(v[i].y - m);
      v[i].z = __expf(v[i].z - m); v[i].w = __expf(v[i].w - m);
      s += row_pick(in(i), (v[i].x + v[i].y) + (v[i].z + v[i].w), 0.f);
    }
    const float inv = 1.0f / G::sum(s, part1);
    float *out = a.y + (uint64_t)r * a.cols;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (in(i)) st4<NT>(out + (i * LANES + lane) * 4, make_float4(v[i].x * inv, v[i].y * inv, v[i].z * inv, v[i].w * inv));
#endif
  }
};

struct LayerNormOp {
  using Args = tally_layernorm_f32_args;
  // (as for the softmax: 80000 x 1500 x 1 261 11.8 / 180 10.4, 60000 x 2048 x 1 212 11.6 / 177 12.5; 200000 x 512 x 3
  // 224 11.5 / 166 11.1, x 4 182 11.3 / 164 13.3; 300000 x 200 x 4 239 11.4 / 170 9.6, x 6 171 10.6 / 171 12.9)
  static uint32_t team_bytes(uint32_t chunk) { return chunk <= 4 ? 48 << 10 : 0; }
  template <class G, uint32_t LANES, int NV, bool NT, bool ONE>
  static __device__ __forceinline__ void row(const Args &a, uint32_t r, uint32_t lane, float4 (&v)[NV],
                                             float *part0, float *part1) {
#ifdef __HIP_DEVICE_COMPILE__
    auto in = [&](int i) { return row_has<LANES, NV>(a.cols, i, lane); };
    float s = 0.f;                                         // (lanes past the end hold zeros)
#pragma unroll
    for (int i = 0; i < NV; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    const float mu = G::sum(s, part0) / (float)a.cols;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const float dx = v[i].x - mu, dy = v[i].y - mu, dz = v[i].z - mu, dw = v[i].w - mu;
      q += row_pick(in(i), (dx * dx + dy * dy) + (dz * dz + dw * dw), 0.f);
    }
    // A single row per group takes ordinary loads here too, the first few of them ahead of the
    // last sum as far as registers go (1557 rows of 1324 columns 4.6 us with buffer loads behind
    // it, 4.45 so; 20000 rows of 1324 / 4096 columns 34.0 / 129.6 and 32.7 / 126.6).
    constexpr int AHEAD = !ONE ? 0 : NV <= 8 ? (NV < 4 ? NV : 4) : 2;
    float4 g0[AHEAD ? AHEAD : 1], b0[AHEAD ? AHEAD : 1];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (in(i)) { g0[i] = ld4<false>(a.gamma + (i * LANES + lane) * 4); b0[i] = ld4<false>(a.beta + (i * LANES + lane) * 4); }
    const float rstd = 1.0f / sqrtf(G::sum(q, part1) / (float)a.cols + a.eps);
    float *out = a.y + (uint64_t)r * a.cols;
    auto norm = [&](int i, float4 gg, float4 bb) {
      return make_float4(__builtin_fmaf((v[i].x - mu) * rstd, gg.x, bb.x), __builtin_fmaf((v[i].y - mu) * rstd, gg.y, bb.y),
                         __builtin_fmaf((v[i].z - mu) * rstd, gg.z, bb.z), __builtin_fmaf((v[i].w - mu) * rstd, gg.w, bb.w));
    };
    if constexpr (ONE) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const uint32_t c = (i * LANES + lane) * 4;
        if (!in(i)) continue;
        if (i < AHEAD) st4<NT>(out + c, norm(i, g0[i < AHEAD ? i : 0], b0[i < AHEAD ? i : 0]));
        else st4<NT>(out + c, norm(i, ld4<false>(a.gamma + c), ld4<false>(a.beta + c)));
      }
    } else {
      const buf_t g = row_buf(a.gamma, 0, a.cols, true), b = row_buf(a.beta, 0, a.cols, true);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const uint32_t byte = (i * LANES + lane) * 16;
        const float4 y = norm(i, buf_ld4<false>(g, byte), buf_ld4<false>(b, byte));
        if (in(i)) st4<NT>(out + byte / 4, y);
      }
    }
#endif
  }
};

// Three kernels per operator, by width: the widest rows a kernel can hold set the registers,
// hence the occupancy, of all of it.  Rows of up to 1024 columns get one that needs a quarter
// of the registers of the next (a high-priority kernel over narrow rows then fits several
// waves per SIMD beside paused best-effort workgroups), rows of up to 4096 the one that the
// operator's footprint is stated for, wider ones the workgroup-wide groups.  WAVES is what the
// original form leaves room for; DEEP instances, which the worker uses for narrow rows, trade
// registers for rows in flight.
template <class Op, int MAXNV, int WAVES, bool DEEP>
struct RowsBodyT {
  using Args = typename Op::Args;
  static constexpr bool TEAMS = MAXNV <= 16;              // (a block of wider rows has more bytes than team_bytes)
  static uint64_t block_bytes(const Args &a) { return 32 * (uint64_t)a.cols; }
  // The rows of several blocks take a worker 3 us and more however narrow they are, longer than 256
  // workers queue at the counter (300000 x 100, 256 x 4, us with the counter alone / in teams 222 / 234;
  // of one block 100000 x 1024, us and us of drain, 312 8.2 / 246 7.3).
  static uint32_t team_bytes(uint32_t workers, uint32_t chunk) {
    return workers >= 512 ? Op::team_bytes(chunk) : chunk == 1 ? 32 << 10 : 0;
  }
  static constexpr int THREADS = kThreads;
  static constexpr int MIN_WAVES = WAVES;
  static constexpr unsigned DYN_LDS = 0;
  static constexpr bool YIELDS = false;
  static constexpr bool RANGE = true;
  static constexpr bool END_BARRIER = false;
  static constexpr uint32_t MAX_COLS = MAXNV * kWave * 4;   // widest row held in registers
  static __device__ __forceinline__ void run(const Args &a, uint32_t bx, uint32_t, uint32_t) { walk<false, true>(a, bx, bx + 1); }
  static __device__ __forceinline__ void run_be(const Args &a, uint32_t bx, uint32_t, uint32_t) { walk<true, true>(a, bx, bx + 1); }
  static __device__ __forceinline__ void run_range(const Args &a, uint32_t first, uint32_t last) { walk<true, false>(a, first, last); }
  template <bool NT, bool ONE>
  static __device__ __forceinline__ void walk(const Args &a, uint32_t first, uint32_t last) {
    const uint32_t r0 = first * 4, want = (last - first) * 4, n = a.rows - r0 < want ? a.rows - r0 : want;
    if constexpr (MAXNV > 16) {
      rows_walk<Op, kThreads, MAXNV / 4, 2, NT>(a, r0, n);
    } else {
      if (a.cols <= 256) rows_walk<Op, kWave, 1, DEEP && !ONE ? 4 : 1, NT, ONE>(a, r0, n);
      else if (a.cols <= 512) rows_walk<Op, kWave, 2, DEEP && !ONE ? 4 : 1, NT, ONE>(a, r0, n);
      else if (a.cols <= 1024) rows_walk<Op, kWave, 4, DEEP && !ONE ? 4 : 1, NT, ONE>(a, r0, n);
      else if constexpr (MAXNV >= 16) {
        if (a.cols <= 2048) rows_walk<Op, kWave, 8, DEEP && !ONE ? (WAVES <= 2 ? 4 : 2) : 1, NT, ONE>(a, r0, n);
        else rows_walk<Op, kWave, 16, DEEP && !ONE && WAVES <= 2 ? 2 : 1, NT, ONE>(a, r0, n);
      }
    }
  }
};
using SoftmaxBody = RowsBodyT<SoftmaxOp, 16, 4, true>;
using SoftmaxNarrowBody = RowsBodyT<SoftmaxOp, 4, 8, false>;
using SoftmaxNarrowDeepBody = RowsBodyT<SoftmaxOp, 4, 4, true>;
using SoftmaxTeamBody = RowsBodyT<SoftmaxOp, 32, 4, true>;
using LayerNormBody = RowsBodyT<LayerNormOp, 16, 2, true>;
using LayerNormNarrowBody = RowsBodyT<LayerNormOp, 4, 8, false>;
using LayerNormNarrowDeepBody = RowsBodyT<LayerNormOp, 4, 4, true>;
using LayerNormTeamBody = RowsBodyT<LayerNormOp, 32, 4, true>;

}  // namespace tally
