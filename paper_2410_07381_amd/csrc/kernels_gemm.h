// bf16 GEMM logical-block body for gfx950: one 256x256 (or 256x128) output tile per logical
// block.
//
// C = A * B with A (m x k) and Bt (n x k) both K-contiguous, so an MFMA operand fragment
// (8 consecutive bf16 along K) is one 16-byte access for either matrix.  Four 64-lane
// waves in a 2x2 arrangement each own a 128x128 sub-tile as 8x8 MFMA 16x16x32 blocks
// (256 fp32 accumulators per lane, which stay in accumulation registers).
//
// What bounds it is how full the one wave of a SIMD keeps its matrix pipe: 131 k cycles of
// MFMA per 256x256x4096 tile.  A first form of this kernel (stages of k = 32, 64-byte row
// pieces, 32x32x16 MFMAs) took 202 k cycles.  Three things were in the way:
//  - half of every cache line: a direct load of 64-byte pieces costs the address unit 16
//    requests per KB, a whole line's 128 bytes 8 (17.3 M L2 requests per 4096^3 product);
//    an LDS stage is therefore k = 64 wide, one line per row;
//  - the epilogue's 2900 vector instructions per wave (16-bit LDS writes): with B as the
//    first MFMA operand a lane holds four neighbouring columns of one row, which leave as
//    one 8-byte LDS write;
//  - a barrier per 1024 cycles with the reads of the next half-step bunched behind it.
// A second one still took 2640 cycles a stage (of 2048 of MFMA) because addresses were computed where
// they were used, in bunches of up to 25 scalar instructions between two MFMAs; with one
// instruction behind each MFMA (see the loop) 1.42 M cycles of 8192^3 became 1.24 M, 0.85 of
// them MFMA.
// In turn on one card, N(0, 1/64) operands, original form, us of the first / second / this state:
// 4096^3 120 / 104 / 98 (bursts of ten), 8192^3 906 (fifty) / 765 / 715 (four; 1.54 PFLOP/s, the
// library 705), 16384 x 12288 x 4096 - / 1172 / 1090, 16384 x 4096 x 16384 - / 1565 / 1460; as
// 256 workers 8192^3 - / 801 / 739.  The clock falls as the pipe fills: 1.69 GHz before, 1.61 now.
//
// LDS holds two stages of both operands (64 KB each, 128 KB in all).  A stage's place is
// refilled as soon as its fragments are in registers, not when its products are done: B's
// after the first half of the stage (the fragments of the second half are read during the
// first), A's six eighths through the second half, so that loads have one to two
// thousand cycles to arrive without a third stage.
//
// Global memory goes straight to LDS (16 bytes per lane, no staging registers).  A stage
// holds 256 rows of 128 bytes; slot chunk c of a row holds k-chunk c xor ((row/2)%8), which
// makes the 16 lanes that a 128-bit LDS read serves together (64 banks, 256 bytes per
// clock) fall into 16 different 16-byte bank groups, without padding.  The lane-to-address
// map of the global side is chosen to produce that layout.
//
// Register budget: the arithmetic VGPRs are kept low on purpose (100 beside the 256
// accumulators) so that waves of a high-priority kernel can become resident beside a
// running tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/tally.h"
#include "kernels_stream.h"
#include "gemm_cover.h"
#include "launch_forms.h"

namespace tally {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

typedef const __attribute__((address_space(1))) void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

// NB = 32-column strips per wave: 4 gives the 256x256 tile, 2 a 256x128 tile (128
// accumulators per lane) for operands whose n is only a multiple of 128.
template <int NB>
struct GemmBodyT {
  static_assert(NB == 2 || NB == 4, "two or four column strips per wave");
  using Args = tally_gemm_bf16_args;
  static constexpr int THREADS = 256;
  static constexpr int MIN_WAVES = 1;
  static constexpr int TILE = 256;                        // rows of C per logical block
  static constexpr int TILE_N = 64 * NB;                  // columns of C per logical block
  static constexpr int KSTEP = 32;                        // k of one MFMA: what k is a multiple of
  static constexpr int BK = 64;                           // k of one LDS stage: 128 bytes of a row
  static constexpr int STAGES = 2;
  static constexpr int MF = 8, NF = 2 * NB;               // 16-row / 16-column blocks of a wave
  static constexpr int LDA_N = 8, LDB_N = 2 * NB;         // direct loads per wave and stage
  static constexpr int OPA = TILE * BK * 2;               // bytes of A in one stage (32 KB)
  static constexpr int OPB = TILE_N * BK * 2;             // bytes of B in one stage
  static constexpr unsigned DYN_LDS = (unsigned)(OPA + OPB) * STAGES;  // 128 KB / 96 KB
  // a tile opens with a barrier that follows the LDS reads of the tile before
  static constexpr bool END_BARRIER = false;
  static constexpr bool YIELDS = true;
  static constexpr bool RANGE = false;
  // share of a tile between two questions for the pause word, `every` k-steps of 32 apart (a stage
  // is two of them and asks once), and the stage after the second, at whose end its answer is
  // acted on; host side, for turnaround estimates
  static double pause_fraction(const Args &a, uint32_t every) {
    const uint32_t nk = a.k / KSTEP, e = (every < 2 ? 2 : every) + 2;
    return nk > e ? (double)e / nk : 1.0;
  }

  static __device__ __forceinline__ void run(const Args &a, uint32_t bx, uint32_t by, uint32_t bz) {
    run_impl<false, false>(a, bx, by, bz, YieldCtl{nullptr, 0, 0, 15, false});
  }
  // best-effort forms: the output tile is written with non-temporal stores (it is not read
  // again by this kernel and would only push other data out of the caches)
  static __device__ __forceinline__ void run_be(const Args &a, uint32_t bx, uint32_t by, uint32_t bz) {
    run_impl<true, false>(a, bx, by, bz, YieldCtl{nullptr, 0, 0, 15, false});
  }
  static __device__ __forceinline__ void run_yielding(const Args &a, uint32_t bx, uint32_t by,
                                                      uint32_t bz, const YieldCtl ctl) {
    run_impl<true, true>(a, bx, by, bz, ctl);
  }

  template <bool NT, bool YIELD>
  static __device__ __forceinline__ void run_impl(const Args &a, uint32_t bx, uint32_t by,
                                                  uint32_t bz, const YieldCtl ctl) {
#ifdef __HIP_DEVICE_COMPILE__  // (buffer resources have no type in the host compiler's pass)
    extern __shared__ __align__(1024) unsigned char tally_dyn_lds[];
    const uint32_t tid = threadIdx.x;
    // (the lane index is made opaque here and again before the epilogue: a worker runs tile
    // after tile, and addresses derived from a plain threadIdx would be kept in registers
    // across the whole worker loop, beyond what a high-priority wave needs free beside it)
    uint32_t lane = tid & 63;
    asm volatile("" : "+v"(lane));
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wm = wave >> 1, wn = wave & 1;
    const uint32_t K = a.k;
    const uint32_t LDA = a.lda ? a.lda : K, LDB = a.ldb ? a.ldb : K;   // row pitches
    const uint32_t nh = K / KSTEP;                        // 32-wide k-steps
    const uint32_t ns = (nh + 1) / 2;                     // stages; the last one may be half full
    const bool half_last = (nh & 1) != 0;

    // Global side of the direct loads.  One load moves 8 rows x 128 bytes to 1 KB of LDS; lane
    // l supplies 16-byte slot l, that is row l/8, k-chunk (l%8) xor ((row/2)%8): for the even
    // loads of a wave that is c = (l%8) xor (l/16), for the odd ones c xor 4.  Buffer
    // addressing: per-lane offsets that never change, one scalar offset per load; the buffers
    // start 4 KB before the tile because the instruction's immediate, which separates the
    // loads of an LDS base, moves the global address too and is taken out again.
    const uint32_t ld_c = (lane & 7) ^ (lane >> 4);
    const uint32_t rowA = wave * 64 + (lane >> 3), rowB = wave * (8 * LDB_N) + (lane >> 3);
    const uint32_t vA0 = (rowA * LDA + ld_c * 8) * 2, vA1 = (rowA * LDA + (ld_c ^ 4) * 8) * 2;
    const uint32_t vB0 = (rowB * LDB + ld_c * 8) * 2, vB1 = (rowB * LDB + (ld_c ^ 4) * 8) * 2;
    // A lane whose offset has its top bit set is outside the buffer: it moves nothing and its
    // slot is filled with zeros.  So are the upper halves of the rows in the last stage of an
    // odd number of k-steps, and whole stages past the last one: the loop below is the same
    // for every stage and needs no peeled ends, whose merging paths cost the compiler copies
    // of the accumulators.
    constexpr uint32_t OOB = 0x80000000u;
    const uint32_t hm0 = (ld_c & 4) ? OOB : 0u, hm1 = hm0 ^ OOB;
    const auto rA = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const unsigned char *)(a.A + bz * a.stride_a + (uint64_t)(by * TILE) * LDA) - 4096),
        0, 0x7fffffff, 0x00027000);
    const auto rB = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const unsigned char *)(a.Bt + bz * a.stride_b + (uint64_t)(bx * TILE_N) * LDB) - 4096),
        0, 0x7fffffff, 0x00027000);
    // scalar offsets of a wave's loads, kept: nothing is computed for one inside the loop
    uint32_t soA[LDA_N], soB[LDB_N];
#pragma unroll
    for (int j = 0; j < LDA_N; ++j) {
      soA[j] = 4096u + (uint32_t)j * 16 * LDA - (uint32_t)(j & 3) * 1024u;
      asm volatile("" : "+s"(soA[j]));
    }
#pragma unroll
    for (int j = 0; j < LDB_N; ++j) {
      soB[j] = 4096u + (uint32_t)j * 16 * LDB - (uint32_t)(j & 3) * 1024u;
      asm volatile("" : "+s"(soB[j]));
    }
    struct Offs { uint32_t even, odd; };
    auto offs = [&](uint32_t v0, uint32_t v1, uint32_t kt) {
      const uint32_t none = kt >= ns ? OOB : 0u, half = (half_last && kt + 1 == ns) ? OOB : 0u;
      return Offs{(v0 + kt * (BK * 2)) | (hm0 & half) | none, (v1 + kt * (BK * 2)) | (hm1 & half) | none};
    };
    // load j of a stage to `at` (the wave's rows of the operand's place in LDS)
    auto load = [&](const auto &r, uint32_t at, const Offs &v, const uint32_t *so, int j) {
      lptr_t l = (lptr_t)(at + (j & 4) * 1024);
      if ((j & 3) == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, l, 16, v.even, so[j], 0, 0);
      if ((j & 3) == 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, l, 16, v.odd, so[j], 1024, 0);
      if ((j & 3) == 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, l, 16, v.even, so[j], 2048, 0);
      if ((j & 3) == 3) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, l, 16, v.odd, so[j], 3072, 0);
    };

    f32x4_t acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Looks at the pause word.  To wait for one is a memory round trip in which the wave's matrix
    // pipe idles and the other three wait at the next barrier (8192^3 as workers 812 us, 757
    // without looks).  So one wave asks with an ordinary load among the operands' and acts on the
    // answer a stage later.  The question goes out between a stage's B and its A: what waits for
    // that B waits for the answer too, a thousand cycles after it was asked, and counts the same
    // loads whether there was one or not.
    uint32_t pause_left = ctl.ticks;   // what is left of this block's pause budget
    uint32_t look = 0;
    const bool looks = YIELD && ctl.ticks != 0 && wave == 0;
    const auto rF = __builtin_amdgcn_make_buffer_rsrc((void *)ctl.flag, 0, 4, 0x00027000);
    auto ask = [&]() { look = __builtin_amdgcn_raw_buffer_load_b32(rF, 0, 0, 16); };   // (sc1)
    auto act = [&]() {
      if (__builtin_amdgcn_readfirstlane(look) == ctl.epoch) yield_while_preempted(ctl, pause_left);
    };
    // stages that ask and those, right after them, that act: never for the other waves
    const uint32_t look_mask = looks ? ctl.mask >> 1 : 0u, ask_at = looks ? look_mask : 1u, act_at = looks ? 0u : 1u;
    // A tile's first loads (every resident tile starts at once after a launch) and its
    // epilogue (32 MiB written by all compute units together) are its heaviest bursts of
    // memory traffic: neither is to start on top of a high-priority kernel.  (The first block
    // of a fetch has just been told by the fetch itself.)
    if (ctl.look_first && looks && nh >= 32) yield_while_preempted(ctl, pause_left);
    // a previous tile's waves may still be reading LDS: fence them off before refilling it
    __syncthreads();
    // LDS as addresses: the operands' places of stage 0, and this wave's rows in the place that the
    // next loads go to
    const uint32_t ldsA = (uint32_t)(uintptr_t)(lptr_t)tally_dyn_lds, ldsB = ldsA + STAGES * OPA;
    uint32_t toA = ldsA + wave * (64 * BK * 2), toB = ldsB + wave * (8 * LDB_N * BK * 2);
    // offsets of the stage whose loads are next: its second half of A's are
    Offs vA = offs(vA0, vA1, 1), vB = offs(vB0, vB1, 1);
    {
      const Offs vb = offs(vB0, vB1, 0), va = offs(vA0, vA1, 0);
#pragma unroll
      for (int j = 0; j < LDB_N; ++j) load(rB, toB, vb, soB, j);
#pragma unroll
      for (int j = 0; j < LDA_N; ++j) load(rA, toA, va, soA, j);
#pragma unroll
      for (int j = 0; j < LDB_N; ++j) load(rB, toB + OPB, vB, soB, j);
#pragma unroll
      for (int j = 0; j < LDA_N / 2; ++j) load(rA, toA + OPA, vA, soA, j);
    }

    // Two B fragment sets (this half-step's and the next one's) and a window of four A fragments;
    // a step is one A fragment against all of B's.  A wave is alone on its SIMD: it issues an
    // instruction every four cycles, so between two MFMAs, 16 cycles apart, three others are free
    // and every further one leaves the matrix pipe idle for four.  So each MFMA is followed by one
    // read, load or address update at most, pinned there, and what can be is kept in registers
    // or updated in place: offsets and LDS addresses move by a stage's k or to the other stage's
    // place with one addition each.  (With addresses computed where they were used, 163 other
    // instructions a stage in bunches of up to 25, a stage took 2640 cycles for its 2048 of
    // MFMAs.)  The MFMAs are inline assembly because the compiler otherwise puts part of the
    // accumulators into arithmetic registers, and so are the updates, which it would sum up anew.
    // Fragment reads: lane l takes row l%16 of a 16-row block and k-chunk 4 kk + l/16
    const uint32_t f_off = (lane & 15) * (BK * 2) + (((lane >> 4) ^ ((lane >> 1) & 7)) * 16);
    uint32_t aK[2], bK[2];                                // addresses of k-halves 0 and 1
    aK[0] = ldsA + wm * (128 * BK * 2) + f_off;
    aK[1] = ldsA + wm * (128 * BK * 2) + (f_off ^ 64);
    bK[0] = ldsB + wn * (16 * NF * BK * 2) + f_off;
    bK[1] = ldsB + wn * (16 * NF * BK * 2) + (f_off ^ 64);
    bf16x8_t fa[4], fb[2][NF];
    typedef const volatile __attribute__((address_space(3))) bf16x8_t *frag_t;   // (volatile: pinned)
    auto read_a = [&](int kk, int i) { fa[(8 * kk + i) & 3] = *(frag_t)(aK[kk] + i * (16 * BK * 2)); };
    auto read_b = [&](int kk, int j) { fb[kk][j] = *(frag_t)(bK[kk] + j * (16 * BK * 2)); };
    auto mma = [&](int kk, int i, int j) {
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                   : "+a"(acc[i][j]) : "v"(fb[kk][j]), "v"(fa[(8 * kk + i) & 3]));
    };
    auto move = [](uint32_t &v, int32_t by) { asm volatile("v_add_u32_e32 %0, %1, %0" : "+v"(v) : "s"(by)); };
    auto flip = [](int32_t &by) { asm volatile("s_sub_i32 %0, 0, %0" : "+s"(by) : : "scc"); };
    auto next_k = [](uint32_t &v) { asm volatile("v_add_u32_e32 %0, 0x80, %0" : "+v"(v)); };
    static_assert(BK * 2 == 0x80, "a stage's k in bytes");
    constexpr int Q = NF / 4;                             // MFMAs between two other instructions

    // stage 0 has landed once only what belongs to stage 1 is in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LDB_N + LDA_N / 2) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_a(0, 0);
#pragma unroll
    for (int j = 0; j < NF; ++j) read_b(0, j);
    read_a(0, 1);
    __builtin_amdgcn_sched_barrier(0);
    int32_t d[2] = {OPA, OPB}, &dA = d[0], &dB = d[NF == MF ? 0 : 1];   // from this stage's place to the other one
    static_assert(NF != MF || OPA == OPB, "one step for both operands");
    toA += OPA;
    uint32_t kt = 0;
    do {
      // first half of the stage; the second half of A's loads of stage kt+1 go out
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) {
          mma(0, i, j);
          if (j == 0 && i < NF) read_b(1, i);
          if (j == Q) {
            if (i + 2 < MF) read_a(0, i + 2);
            else read_a(1, i + 2 - MF);
          }
          if (j == 2 * Q && i < LDA_N / 2) load(rA, toA, vA, soA, LDA_N / 2 + i);
          if (j == 3 * Q) {
            if (i == 0) move(bK[0], dB);
            if (i == 1) next_k(vB.even);
            if (i == 2) next_k(vB.odd);
            if (i == 3) asm volatile("s_sub_i32 %0, %0, %1" : "+s"(toA) : "s"(dA) : "scc");
            if (i == 4) next_k(vA.even);
            if (i == 5) next_k(vA.odd);
            if (i == 6) move(aK[0], dA);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      // From here on it is stage kt+2 that is loaded: the last one, or one that does not exist
      if (__builtin_expect(kt + 3 >= ns, 0)) {
        const uint32_t m0 = kt + 3 == ns ? (half_last ? hm0 : 0u) : OOB, m1 = kt + 3 == ns ? (half_last ? hm1 : 0u) : OOB;
        vA.even |= m0; vA.odd |= m1; vB.even |= m0; vB.odd |= m1;
      }
      // second half.  B of stage kt+1 is in LDS for everyone; everyone is done with B of stage
      // kt, whose place takes the loads of stage kt+2
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(1)" ::"n"(LDA_N) : "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MF; ++i) {
        if (i == MF - 2) {
          // the same for A
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)" ::"n"(LDB_N), "n"(NF > 5 ? 1 : 0) : "memory");
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < NF; ++j) {
          mma(1, i, j);
          if (j == 0) {
            if (i + 2 < MF) read_a(1, i + 2);
            else read_a(0, i + 2 - MF);
          }
          if constexpr (YIELD) {
            // (one wave pauses, the others meet it at the next barrier)
            if (i == MF - 2 && j == Q - 1) {
              if (__builtin_expect((kt & look_mask) == act_at, 0)) act();
              if (__builtin_expect((kt & look_mask) == ask_at, 0)) ask();
            }
          }
          if (j == Q && i < NF) read_b(0, i);
          if (j == 2 * Q) {
            if (i < 4) load(rB, toB, vB, soB, LDB_N > 4 ? 2 * i : i);
            if (i >= MF - 2) load(rA, toA, vA, soA, 2 * (i - (MF - 2)));
            if (i == 4) move(bK[1], dB);
            if (i == 5) move(aK[1], dA);
          }
          if (j == 3 * Q) {
            if (i < 4 && LDB_N > 4) load(rB, toB, vB, soB, 2 * i + 1);
            if (i >= MF - 2) load(rA, toA, vA, soA, 2 * (i - (MF - 2)) + 1);
            if (i == 4) asm volatile("s_add_i32 %0, %0, %1" : "+s"(toB) : "s"(dB) : "scc");
            if (i == 5) flip(d[0]);
            if (i == 5 && NF != MF) flip(d[1]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } while (++kt < ns);
    // what was still on its way is the zeros of stages past the last one
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // Before the epilogue: the last answer, where its question is at most four stages old; where questions
    // are further apart, or the tile was shorter than their distance, the word is read again (a wait of
    // 0.7 us, once in a tile).
    if (looks && nh >= 32) {
      if (look_mask < 4) act();
      else yield_while_preempted(ctl, pause_left);
    }
    // every wave is past its last fragment read: LDS can be reused as staging space
    __syncthreads();
    // The accumulators are read below through inline assembly, which the compiler's
    // hazard recogniser cannot see into: keep the last MFMAs from being interleaved with
    // those reads and give the matrix pipe time to retire its last results first.
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // Epilogue.  B was the first MFMA operand, so lane l, register r of block (i, j) holds
    // row 16 i + l%16, column 16 j + 4 (l/16) + r: four neighbours of one row, packed to 8
    // bytes with two hardware conversions (round to nearest even).  Each wave stages its
    // 128 x 16 NF sub-tile through a region of LDS of its own (16-byte chunks xor-swizzled by
    // the row, so that neither the 8-byte writes nor the 16-byte reads conflict) and writes
    // whole row pieces, 16 bytes per lane.  Each accumulator is read where it is used: a
    // wholesale copy of the accumulators into arithmetic registers would double the wave's
    // register footprint, which decides how many other waves fit beside this one.
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    constexpr uint32_t ROWB = 32 * NF;                    // bytes of a sub-tile row (256 / 128)
    constexpr uint32_t LPR = ROWB / 16;                   // chunks (and lanes reading back) per row
    constexpr uint32_t RPI = 64 / LPR;                    // rows per wave instruction
    asm volatile("" : "+v"(lane));
    auto swz = [](uint32_t row) { return NF == 8 ? (row & 15) : ((row >> 1) & 7); };
    unsigned char *stage = tally_dyn_lds + wave * (128 * ROWB);
    const uint32_t w_row = lane & 15, w_sw = (lane >> 5) ^ swz(w_row);
    unsigned char *w_base = stage + w_row * ROWB + ((lane >> 4) & 1) * 8;
    const uint32_t r_row = lane / LPR, r_chunk = lane % LPR;
    uint16_t *gC = a.C + bz * a.stride_c + (uint64_t)(by * TILE + wm * 128) * a.n + bx * TILE_N + wn * (16 * NF);
    const uint32_t g_off = r_row * a.n + r_chunk * 8;
    // an output too large to stay in the 256 MB Infinity Cache beside anything else is
    // written with non-temporal stores in the original form too (2 GB of attention scores:
    // 960 us -> 620 us)
    const bool big_output = (uint64_t)a.m * a.n * a.batch * 2u > kGemmBigOutput;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int ii = 0; ii < MF / 2; ++ii)
#pragma unroll
        for (int j = 0; j < NF; ++j) {
          const int i = h * (MF / 2) + ii;
          float v0, v1, v2, v3;
          asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v0) : "a"(acc[i][j][0]));
          asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v1) : "a"(acc[i][j][1]));
          asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v2) : "a"(acc[i][j][2]));
          asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v3) : "a"(acc[i][j][3]));
          const f32x2_t p0 = {v0, v1}, p1 = {v2, v3};
          uint2 w;
          w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(p0, bf16x2_t));
          w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(p1, bf16x2_t));
          *reinterpret_cast<uint2 *>(w_base + i * (16 * ROWB) + ((w_sw ^ (2 * j)) * 16)) = w;
        }
#pragma unroll
      for (uint32_t t = h * (64 / RPI); t < (h + 1) * (64 / RPI); ++t) {
        const uint32_t row = t * RPI + r_row;
        const uint4 v = *reinterpret_cast<const uint4 *>(stage + row * ROWB + ((r_chunk ^ swz(row)) * 16));
        uint16_t *g = gC + (uint64_t)(t * RPI) * a.n + g_off;
        if (NT || big_output) {
          const u32x4_nt w = {v.x, v.y, v.z, v.w};
          __builtin_nontemporal_store(w, reinterpret_cast<u32x4_nt *>(g));
        } else {
          *reinterpret_cast<uint4 *>(g) = v;
        }
      }
    }
#endif
  }
};
using GemmBody = GemmBodyT<4>;
using GemmN128Body = GemmBodyT<2>;

// Blocks of 16x16 next to one another in a row of blocks, from column col0 on, to C.  B was the first MFMA
// operand, so lane l, register r of a block holds row l%16, column 4 (l/16) + r: four neighbours of one row,
// packed to 8 bytes.  Of two column blocks the swaps make eight neighbours per lane (group l/16 columns 8 (l/16)
// .. +7 of the 32), so that whole 64-byte pieces leave (4352 x 4864 x 64 13.3 us; 18.8 as 32-byte pieces).
// NT: past the caches, for outputs whose rows all start at 16 bytes and have no remainder.
template <bool NAN7FC0, bool NT, int RB>
__device__ __forceinline__ void store_blocks(const tally_gemm_bf16_args &a, uint32_t bz, uint32_t row, uint32_t col0,
                                             uint32_t lane, const f32x4_t (&acc)[RB]) {
#ifdef __HIP_DEVICE_COMPILE__
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  auto pack = [](float x, float y) {
    if constexpr (NAN7FC0) return f32_to_bf16(x) | (uint32_t)f32_to_bf16(y) << 16;
    const f32x2_t p = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, bf16x2_t));
  };
  auto store = [&](auto wide, int j) {                     // `wide` blocks from j on
    constexpr int W = decltype(wide)::value;
    uint32_t w[2 * W];
#pragma unroll
    for (int e = 0; e < W; ++e) {
      w[2 * e] = pack(acc[j + e][0], acc[j + e][1]);
      w[2 * e + 1] = pack(acc[j + e][2], acc[j + e][3]);
    }
    if constexpr (W == 2) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
        asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(w[q]), "+v"(w[2 + q]));
    }
    const uint32_t col = col0 + 16 * j + (lane >> 4) * (4 * W);
    uint16_t *g = a.C + bz * a.stride_c + (uint64_t)row * a.n + col;
    if constexpr (NT) {
      static_assert(W == 2, "16 bytes");
      __builtin_nontemporal_store(u32x4_nt{w[0], w[1], w[2], w[3]}, reinterpret_cast<u32x4_nt *>(g));
    } else if (row < a.m) {
      if (col + 4 * W <= a.n) {
        // (rows start at any multiple of 2 bytes and are stored alike: 413 x 741 x 640 x 12 in 19.0 us,
        // 23.5 with the widest aligned stores that each row allows)
        __builtin_memcpy(g, w, 8 * W);
      } else {
#pragma unroll
        for (int e = 0; e < 4 * W; ++e)
          if (col + e < a.n) g[e] = (uint16_t)(w[e / 2] >> (16 * (e & 1)));
      }
    }
  };
#pragma unroll
  for (int j = 0; j + 1 < RB; j += 2) store(std::integral_constant<int, 2>{}, j);
  if constexpr (RB & 1) store(std::integral_constant<int, 1>{}, RB - 1);
#endif
}

// The same operator with smaller tiles and predicated edges: (32 RA) x (32 RB) outputs per
// workgroup, four waves in a 2x2 arrangement of RA x RB blocks of 16x16 each.  32x32 is the
// logical block of the small or ragged GEMM (the high-priority inference-like layer, whose grid
// is often far smaller than the GPU and where every kernel is a chain of memory latencies);
// 32x64, 64x64 and 128x64 cover its original form where the 32x32 tiles are more than the
// compute units, and the large tile's where there are too few of those, beside best-effort jobs
// and where K is short (see gemm_cover).
//
// Every tile of every size, the 256-row tiles included, adds its products in the same order:
// one accumulator per output, k ascending, one 16x16x32 MFMA per 32 of it with B first, one
// rounding at the end.  The bits of a product depend neither on the form it runs in
// nor on where a job was stopped and resumed.  (An earlier 32x32 tile split K between its waves:
// a job finished in its parts, or run in the original form, came out in other bits.)
//
// Operands are loaded as whole 128-byte lines, 8 rows per load (8 requests per KB; a load in
// fragment shape costs one per lane), AHEAD stages of 64 k ahead in registers, and shared by the
// four waves through LDS.  What bounds the two smallest tiles is the serial chain of short
// stages, and LDS (every operand byte is read twice: 192 cycles per stage of a 32x32 tile): they
// have two LDS buffers, so that the fragments of one are read while the other is written and a
// stage has one barrier.  The larger two have room for one buffer and take two barriers.
// Within 128 registers and 31 KB of LDS: what a resident 256x256 tile leaves free, since a
// high-priority kernel that does not fit beside the paused tiles of a best-effort GEMM waits for
// them.
//
// us for 32x32 / 32x64 / 64x64 / 128x64: 128 x 768 x 3072 (96 tiles of 32x32) 7.7 / 10.7 / 16.5;
// 128 x 3072 x 768 (384) 5.3 / 4.8 / 5.8; 1000 x 2300 x 768 13.9 / 12.0 / 10.5 / 11.7;
// 512 x 4096 x 4096 53 / 39 / 29 / 32; 2048 x 4096 x 4096 195 / 140 / 101 / 85 (0.81 PFLOP/s).
// With K split between the waves of the 32x32 tile: 7.7, 5.0, 15.1, 50 and 199.
//
// NAN7FC0: a NaN leaves as 0x7FC0, which is what the ragged GEMM has always written; those with
// blocks of 256 rows write what the hardware's conversion makes of the MFMA's NaN (0xFFC0).
template <int RA, int RB, bool NAN7FC0 = false>
struct GemmTileT {
  using Args = tally_gemm_bf16_args;
  static constexpr int THREADS = 256;
  static constexpr int MIN_WAVES = 4;
  static constexpr unsigned DYN_LDS = 0;
  static constexpr bool YIELDS = true;
  static constexpr bool RANGE = false;
  // a block's last barrier follows its last fragment read
  static constexpr bool END_BARRIER = false;
  static constexpr uint32_t TM = 32 * RA, TN = 32 * RB;
  static constexpr int LA = RA, LB = RB;                  // loads of a wave and stage
  static constexpr bool TWO = RA * RB <= 2;               // LDS holds two stages
  static constexpr int AHEAD = RA * RB == 1 ? 8 : RA * RB <= 2 ? 4 : RA * RB <= 4 ? 2 : 1;
  static constexpr int ROUND = TWO ? AHEAD : 16 / (RA * RB);   // stages between two looks at the pause word, at least
  static constexpr uint32_t SA = TM * 128, STAGE = (TM + TN) * 128;   // bytes of A, of both in a stage
  // share of a tile between asking for the pause word and pausing on the answer to the next
  // question, `every` k-steps of 32 apart (see look_round); host side, for turnaround estimates
  static double pause_fraction(const Args &a, uint32_t every) {
    const uint32_t ns = (a.k + 63) / 64, apart = every / 2 > ROUND ? every / 2 : ROUND;
    return ns > apart + ROUND ? (double)(apart + ROUND) / ns : 1.0;
  }

  static __device__ __forceinline__ void run(const Args &a, uint32_t bx, uint32_t by, uint32_t bz) {
    run_impl<false>(a, bx, by, bz, YieldCtl{nullptr, 0, 0, 15, false});
  }
  static __device__ __forceinline__ void run_be(const Args &a, uint32_t bx, uint32_t by, uint32_t bz) { run(a, bx, by, bz); }
  static __device__ __forceinline__ void run_yielding(const Args &a, uint32_t bx, uint32_t by, uint32_t bz, const YieldCtl ctl) {
    run_impl<true>(a, bx, by, bz, ctl);
  }
  template <bool YIELD>
  static __device__ __forceinline__ void run_impl(const Args &a, uint32_t bx, uint32_t by, uint32_t bz, const YieldCtl ctl) {
    __shared__ __align__(16) unsigned char s_ab[STAGE * (TWO ? 2 : 1)];
    // (with one or two stages the loads of six more that do not exist would be most of the work)
    if (AHEAD > 2 && a.k <= 128) run_ahead<2, YIELD>(a, s_ab, bx, by, bz, ctl);
    else run_ahead<AHEAD, YIELD>(a, s_ab, bx, by, bz, ctl);
  }
  // SETS stages of operands on their way in registers
  template <int SETS, bool YIELD>
  static __device__ __forceinline__ void run_ahead(const Args &a, unsigned char *s_ab, uint32_t bx, uint32_t by, uint32_t bz,
                                                   const YieldCtl ctl) {
#ifdef __HIP_DEVICE_COMPILE__  // (buffer resources have no type in the host compiler's pass)
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // (a worker keeps no addresses across its tiles)
    const uint32_t lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wm = wave >> 1, wn = wave & 1;
    const uint32_t K = a.k;
    const uint32_t LDA = a.lda ? a.lda : K, LDB = a.ldb ? a.ldb : K;
    const uint32_t ns = (K + 63) / 64;

    // A load moves 8 rows, lane l the 16-byte piece l%8 of row l/8.  A lane whose offset has its
    // top bit set is outside the buffer and gets zeros: rows past the matrix, pieces past K in
    // the last stage (K is a multiple of 32), stages past the last one.
    constexpr uint32_t OOB = 0x80000000u;
    const uint32_t r8 = lane >> 3, p8 = lane & 7;
    const buf_t rA = make_buf(a.A + bz * a.stride_a + (uint64_t)by * TM * LDA, 0x7fffffffu);
    const buf_t rB = make_buf(a.Bt + bz * a.stride_b + (uint64_t)bx * TN * LDB, 0x7fffffffu);
    uint32_t vA[LA], vB[LB];
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const uint32_t r = (wave * LA + j) * 8 + r8;
      vA[j] = by * TM + r < a.m ? (r * LDA + p8 * 8) * 2 : OOB;
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const uint32_t r = (wave * LB + j) * 8 + r8;
      vB[j] = bx * TN + r < a.n ? (r * LDB + p8 * 8) * 2 : OOB;
    }
    const uint32_t half = (K & 32) && (p8 & 4) ? OOB : 0u;
    struct Set { uint4 a[LA], b[LB]; };
    auto request = [&](Set &s, uint32_t c) {
      const uint32_t none = (c >= ns ? OOB : 0u) | (c + 1 == ns ? half : 0u);
      const uint32_t so = __builtin_amdgcn_readfirstlane(c >= ns ? 0u : c * 128);
#pragma unroll
      for (int j = 0; j < LA; ++j) s.a[j] = buf_ld16(rA, vA[j] | none, so);
#pragma unroll
      for (int j = 0; j < LB; ++j) s.b[j] = buf_ld16(rB, vB[j] | none, so);
    };
    // piece p of row r lies at slot p xor ((r/2)%8): the 16 lanes that a 128-bit access serves
    // together fall into 16 different 16-byte bank groups, writing and reading
    const uint32_t w_off = r8 * 128 + (p8 ^ (r8 >> 1)) * 16;               // slot xor 4 in odd groups of 8 rows
    auto store = [&](const Set &s, uint32_t buf) {
#pragma unroll
      for (int j = 0; j < LA; ++j) {
        const uint32_t g = wave * LA + j;
        *reinterpret_cast<uint4 *>(s_ab + buf * STAGE + g * 1024 + (w_off ^ ((g & 1) * 64))) = s.a[j];
      }
#pragma unroll
      for (int j = 0; j < LB; ++j) {
        const uint32_t g = wave * LB + j;
        *reinterpret_cast<uint4 *>(s_ab + buf * STAGE + SA + g * 1024 + (w_off ^ ((g & 1) * 64))) = s.b[j];
      }
    };
    // lane l takes row l%16 of a 16-row block, k-chunk 4 kk + l/16
    const uint32_t f_off = (lane & 15) * 128 + (((lane >> 4) ^ ((lane >> 1) & 7)) * 16);
    const uint32_t fA = wm * (16 * RA * 128) + f_off, fB = SA + wn * (16 * RB * 128) + f_off;
    auto read = [&](uint32_t buf, uint32_t at, int kk, int i) {
      return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(s_ab + buf * STAGE + (at ^ (kk * 64)) + i * 2048));
    };
    f32x4_t acc[RA][RB];
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
      for (int j = 0; j < RB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    Set s[SETS];
#pragma unroll
    for (int d = 0; d < SETS; ++d) {
      request(s[d], d);
      __builtin_amdgcn_sched_barrier(0);                  // (in the order in which they are waited for)
    }
    if constexpr (TWO) {
      store(s[0], 0);
      request(s[0], SETS);
      __syncthreads();
    }
    // Looks at the pause word.  Waiting for one costs the workgroup 0.7 us, several of its stages:
    // one lane asks for the word at the start of a round of STEPS stages, behind the loads on their
    // way, and has it at the start of the next.  (Its offset, not a branch, says who asks and
    // when: all others are outside the buffer.)
    constexpr int STEPS = YIELD && SETS == AHEAD ? ROUND : SETS;
    uint32_t pause_left = ctl.ticks, look = 0;
    const buf_t rF = make_buf(ctl.flag, YIELD && ctl.ticks != 0 ? 4 : 0);
    const uint32_t v_look = tid == 0 ? 0u : OOB, look_mask = (ctl.mask >> 1) & ~(STEPS - 1u);   // in stages
    auto look_round = [&](uint32_t c) {
      if constexpr (YIELD) {
        // one wave pauses; the others meet it at the next barrier
        if (__builtin_amdgcn_readfirstlane(look) == ctl.epoch) yield_while_preempted(ctl, pause_left);
        look = __builtin_amdgcn_raw_buffer_load_b32(rF, v_look | ((c & look_mask) == look_mask ? 0u : OOB), 0, 16);  // (sc1)
      }
    };
    // stage c, whose operands (with two buffers those of stage c + 1) are in set d
    auto step = [&](int d, uint32_t c) {
      bf16x8_t fa[2][RA], fb[2][RB];
      if constexpr (TWO) {
        static_assert(SETS % 2 == 0, "the buffer is that of the set");
        const int next = (d + 1) % SETS;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
          for (int j = 0; j < RB; ++j) fb[kk][j] = read(d & 1, fB, kk, j);
#pragma unroll
          for (int i = 0; i < RA; ++i) fa[kk][i] = read(d & 1, fA, kk, i);
        }
        store(s[next], (d + 1) & 1);
        request(s[next], c + 1 + SETS);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        store(s[d], 0);
        request(s[d], c + SETS);
        __syncthreads();
        // (fragments are read ahead of the products, not one by one between them)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
          for (int j = 0; j < RB; ++j) fb[kk][j] = read(0, fB, kk, j);
#pragma unroll
          for (int i = 0; i < RA; ++i) fa[kk][i] = read(0, fA, kk, i);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
          for (int j = 0; j < RB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[kk][j], fa[kk][i], acc[i][j], 0, 0, 0);
      __syncthreads();
    };
    // Rounds of STEPS stages, then what is left of one: no way out of the middle of the loop, which
    // the compiler would give an edge back to its head and with it a wait for every load there.
    uint32_t c = 0;
    for (; c + STEPS <= ns; c += STEPS) {
      look_round(c);
#pragma unroll
      for (int d = 0; d < STEPS; ++d) step(d % SETS, c + d);
    }
    auto rest = [&](auto &&self, auto at) -> void {
      constexpr int d = decltype(at)::value;
      if constexpr (d + 1 < STEPS)
        if (c + d < ns) {
          step(d % SETS, c + d);
          self(self, std::integral_constant<int, d + 1>{});
        }
    };
    rest(rest, std::integral_constant<int, 0>{});
#pragma unroll
    for (int i = 0; i < RA; ++i)
      store_blocks<NAN7FC0, false>(a, bz, by * TM + (wm * RA + i) * 16 + (lane & 15), bx * TN + wn * 16 * RB, lane, acc[i]);
#endif
  }
};
using GemmTile32 = GemmTileT<1, 1>;

// The same operator in tiles of one wave, (16 NA) x (16 NB), for outputs of so few tiles that what bounds them
// is how a stage's instructions follow one another.  A tile that takes its operands through registers writes
// them to LDS, and a 16-byte write takes a wave 35 cycles and the unit 13 (a read 17 and 4, a direct load 16
// on the unit); here they go straight to LDS, R stages of 64 k ahead, in the large tile's layout.  LDS serves
// a wave in order and nobody else writes there, so there is no barrier: a stage waits for the next one's loads,
// reads its fragments, asks for the stage that takes its own place and multiplies.
// R is what 24 KB hold (31 KB are free beside a resident 256x256 tile, and 28 KB are no faster); with fewer the
// loads' latency shows (16x16, 128 x 768 x 3072, R = 6 / 4 / 3: 6.1 / 7.8 / 10.9 us).  The order of the products is that of every tile.
// us through registers (16x16 of one wave, 32x32 or 32x64, the best) / so, operands from the Infinity Cache:
// 128 x 768 x 3072 7.7 / 6.1, 128 x 768 x 768 3.7 / 3.2, 128 x 2304 x 768 4.9 / 4.1, 128 x 3072 x 768 4.9 / 4.2,
// 48 x 2048 x 3072 7.7 / 6.3, 100 x 1000 x 1536 5.3 / 4.2, 256 x 1024 x 768 4.0 / 3.8, 33 x 5000 x 768 5.1 / 4.0.
//
// Tiles of one column of tiles share a panel of B, tiles of one row a panel of A.  The longer side of the output
// is what has many panels, and each die takes a run of those, so that it reads its share of the larger operand and
// all of the smaller one.  Workgroups go to the dies in turn, hence a grid of (8, tiles of a panel, panels of a die);
// the panels of a batch follow one another.  us with columns dealt out to the dies whatever the shape (those of a
// batch in a plain grid) / so, operands from the caches and from memory: 8192 x 16 x 1536 21.7 / 4.0 and 27.6 / 6.6,
// 2048 x 64 x 4096 15.2 / 7.0 and 16.4 / 10.3, 512 x 128 x 1536 3.9 / 3.8 and 4.2 / 3.9,
// 12 of 112 x 73 x 1696 7.8 / 4.3 and 8.3 / 6.1; with columns along the grid's first extent 100 x 1000 x 3072 8.8 / 6.6.
template <int NA, int NB, bool NAN7FC0 = false>
struct GemmWaveT {
  using Args = tally_gemm_bf16_args;
  static_assert(NA * NB <= 2, "one or two blocks");
  static constexpr int THREADS = 64;
  static constexpr int MIN_WAVES = 4;
  static constexpr uint32_t TM = 16 * NA, TN = 16 * NB;
  static constexpr int LA = 2 * NA, LB = 2 * NB, L = LA + LB;   // loads of a stage
  static constexpr int R = NA * NB == 1 ? 6 : 4;
  static constexpr uint32_t SA = TM * 128, STAGE = SA + TN * 128;
  // (dynamic: the compiler gives a kernel that LDS lets on a SIMD only twice a third of its registers, whatever
  // it uses, and 176 do not fit beside a resident tile's 352)
  static constexpr unsigned DYN_LDS = STAGE * R;
  static dim3 grid(const Args &a) {
    const uint32_t x = (a.n + TN - 1) / TN, y = (a.m + TM - 1) / TM;
    return dim3(8, a.m > a.n ? x : y, ((a.m > a.n ? y : x) * a.batch + 7) / 8);
  }
  static __device__ __forceinline__ void run(const Args &a, uint32_t die, uint32_t in, uint32_t at) {
#ifdef __HIP_DEVICE_COMPILE__  // (buffer resources have no type in the host compiler's pass)
    extern __shared__ __align__(1024) unsigned char tally_dyn_lds[];
    uint32_t bx, by, bz;
    if (!wave_tile(a, TM, TN, die, in, at, &bx, &by, &bz)) return;
    const uint32_t lane = threadIdx.x;
    const uint32_t K = a.k;
    const uint32_t LDA = a.lda ? a.lda : K, LDB = a.ldb ? a.ldb : K;
    const uint32_t ns = (K + 63) / 64;
    // A load moves 8 rows x 128 bytes to 1 KB of LDS; lane l supplies 16-byte slot l, that is row l/8, k-chunk
    // (l%8) xor ((row/2)%8).  A lane whose offset has its top bit set is outside the buffer and its slot is
    // filled with zeros: rows past the matrix, k past K in a last stage that is half full.
    constexpr uint32_t OOB = 0x80000000u;
    const buf_t rA = make_buf(a.A + bz * a.stride_a + (uint64_t)by * TM * LDA, 0x7fffffffu);
    const buf_t rB = make_buf(a.Bt + bz * a.stride_b + (uint64_t)bx * TN * LDB, 0x7fffffffu);
    const uint32_t r8 = lane >> 3, c8 = (lane & 7) ^ (lane >> 4);   // (odd groups of 8 rows: c8 xor 4)
    uint32_t vA[LA], vB[LB];
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const uint32_t r = j * 8 + r8;
      vA[j] = by * TM + r < a.m ? (r * LDA + (c8 ^ ((j & 1) * 4)) * 8) * 2 : OOB;
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const uint32_t r = j * 8 + r8;
      vB[j] = bx * TN + r < a.n ? (r * LDB + (c8 ^ ((j & 1) * 4)) * 8) * 2 : OOB;
    }
    const uint32_t base = (uint32_t)(uintptr_t)(lptr_t)tally_dyn_lds, end = base + R * STAGE;
    uint32_t to = base, so = 0, left = ns;                 // the next stage to ask for: its place, its k in bytes, how many
    auto request = [&]() {
      if (--left == 0 && (K & 32)) {
        const uint32_t h0 = c8 & 4 ? OOB : 0u, h1 = h0 ^ OOB;
#pragma unroll
        for (int j = 0; j < LA; ++j) vA[j] |= j & 1 ? h1 : h0;
#pragma unroll
        for (int j = 0; j < LB; ++j) vB[j] |= j & 1 ? h1 : h0;
      }
#pragma unroll
      for (int j = 0; j < LA; ++j) __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (lptr_t)(to + j * 1024), 16, vA[j], so, 0, 0);
#pragma unroll
      for (int j = 0; j < LB; ++j) __builtin_amdgcn_raw_ptr_buffer_load_lds(rB, (lptr_t)(to + SA + j * 1024), 16, vB[j], so, 0, 0);
      so += 128;
      to = to + STAGE == end ? base : to + STAGE;
    };
    // lane l takes row l%16 of a 16-row block, k-chunk 4 kk + l/16; two sets, this stage's and the next one's
    const uint32_t f_off = (lane & 15) * 128 + (((lane >> 4) ^ ((lane >> 1) & 7)) * 16);
    typedef const volatile __attribute__((address_space(3))) bf16x8_t *frag_t;   // (volatile: pinned)
    bf16x8_t fa[2][2][NA], fb[2][2][NB];
    uint32_t from = base;                                  // place of the next stage to read
    auto read = [&](int f) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const uint32_t at = from + (f_off ^ (kk * 64));
#pragma unroll
        for (int j = 0; j < NB; ++j) fb[f][kk][j] = *(frag_t)(at + SA + j * 2048);
#pragma unroll
        for (int i = 0; i < NA; ++i) fa[f][kk][i] = *(frag_t)(at + i * 2048);
      }
      from = from + STAGE == end ? base : from + STAGE;
    };
    f32x4_t acc[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int f) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[f][kk][j], fa[f][kk][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    // A stage whose fragments have been asked for: once they are here its place is free, and once only R - 2
    // stages are on their way the next one has landed.
    auto step = [&](int f) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(L * (R - 2)) : "memory");
      read(f ^ 1);
      request();
      multiply(f);
    };
    // the last R stages, AFTER of them behind this one: nothing is asked for any more
    auto finish = [&](auto &&self, auto after, auto set) -> void {
      constexpr int AFTER = decltype(after)::value, f = decltype(set)::value;
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(AFTER ? L * (AFTER - 1) : 0) : "memory");
      if constexpr (AFTER > 0) read(f ^ 1);
      multiply(f);
      if constexpr (AFTER > 0) self(self, std::integral_constant<int, AFTER - 1>{}, std::integral_constant<int, f ^ 1>{});
    };
    if (ns >= (uint32_t)R) {
#pragma unroll
      for (int d = 0; d < R; ++d) request();
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L * (R - 1)) : "memory");
      read(0);
      uint32_t pairs = (ns - R) / 2;
      if ((ns - R) & 1) {
        step(0);
        for (; pairs; --pairs) { step(1); step(0); }
        finish(finish, std::integral_constant<int, R - 1>{}, std::integral_constant<int, 1>{});
      } else {
        for (; pairs; --pairs) { step(0); step(1); }
        finish(finish, std::integral_constant<int, R - 1>{}, std::integral_constant<int, 0>{});
      }
    } else {
      for (uint32_t d = 0; d < ns; ++d) request();
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      for (uint32_t d = 0; d < ns; ++d) {
        read(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        multiply(0);
      }
    }
#pragma unroll
    for (int i = 0; i < NA; ++i)
      store_blocks<NAN7FC0, false>(a, bz, by * TM + i * 16 + (lane & 15), bx * TN, lane, acc[i]);
#endif
  }
};
// The same operator in tiles of (32 RA) x (32 RB), four waves in a 2x2 arrangement, whose operands go straight to
// LDS, R stages of 64 k ahead in a ring, in the large tile's layout: for products between a few small tiles and
// one 256x128 tile per compute unit, where nobody else needs the LDS (the tiles above are for those beside
// best-effort workgroups).  Fragments are read a stage ahead, so that a stage has one barrier and a wave, alone on
// its SIMD or one of two there, finds a read or a load to issue behind every MFMA.
// What bounds it is what the compute unit brings in: a KB of operands takes 16 cycles to load to LDS, and 4 for
// each of the two waves that read it, which is 96 (RA + RB) cycles a stage, against 32 RA RB of MFMA a wave: at
// 128x128 768 and 512 (measured 810; 64x64 430 for 384).  Hence the times below, about 2.5 us and those stages.
// The last R stages ask for nothing any more (as loads outside the buffers, which take as long as others, they were
// 0.5 us of every tile).
// us in tiles through registers, the best of 32x64, 64x64 and 128x64 / so, operands from the Infinity Cache:
// 400 x 1200 x 2048 9.9 / 7.0 (32x64), 1024 x 1024 x 2048 12.0 / 8.4 (64x64), 1000 x 1500 x 2048 16.5 / 9.9 (64x96),
// 1500 x 1500 x 2048 22.0 / 13.7 (96x96), 1024 x 2048 x 2048 16.8 / 11.6 (128x64), 1000 x 2300 x 768 10.6 / 7.6 (128x96),
// 512 x 6144 x 4096 43.1 / 26.1 (128x96), 2048 x 2048 x 2048 25.8 / 18.0 (128x128; 24.1 in 256x128).
//
// Workgroups go to the eight dies in turn.  Each die takes a run of tiles in an order that makes it a patch: bands
// of H rows of tiles, column after column; the products of a batch follow one another, so that the dies' shares
// differ by one tile (12 of 100 x 900 x 768 6.1 us, 13.4 with every product's remainder on the same dies).
template <int RA, int RB, int R, bool NAN7FC0 = false>
struct GemmRingT {
  using Args = tally_gemm_bf16_args;
  static constexpr int THREADS = 256;
  static constexpr uint32_t TM = 32 * RA, TN = 32 * RB;
  static constexpr int L = RA + RB;                       // loads of a wave and stage
  static constexpr uint32_t SA = TM * 128, STAGE = SA + TN * 128;
  static constexpr unsigned DYN_LDS = STAGE * R;
  static constexpr int MIN_WAVES = 160 * 1024 / DYN_LDS;
  static constexpr bool YIELDS = true;
  // stages between two looks at the pause word, at least, which is also how long a look takes (R - 2 stages after it
  // the operands asked for before it have to be there anyway)
  static constexpr int ROUND = RA * RB >= 8 ? 2 : 4;
  // share of a tile between asking for the pause word and pausing on the answer to the next question, or the end of
  // the tile (see look_round); host side, for turnaround estimates
  static double pause_fraction(const Args &a, uint32_t every) {
    const uint32_t ns = (a.k + 63) / 64, apart = every / 2 > ROUND ? every / 2 : ROUND;
    return ns > apart + ROUND ? (double)(apart + ROUND) / ns : 1.0;
  }
  static uint32_t groups(const Args &a) {                 // (as many for every die)
    return (((a.n + TN - 1) / TN) * ((a.m + TM - 1) / TM) * a.batch + 7) / 8 * 8;
  }
  static __device__ __forceinline__ void run(const Args &a, uint32_t id, uint32_t, uint32_t) {
#ifdef __HIP_DEVICE_COMPILE__  // (buffer resources have no type in the host compiler's pass)
    uint32_t bx, by, bz;
    if (!ring_tile(a, TM, TN, id, &bx, &by, &bz)) return;
    run_tile<false>(a, bx, by, bz, YieldCtl{nullptr, 0, 0, 15, false});
#endif
  }
  static __device__ __forceinline__ void run_yielding(const Args &a, uint32_t bx, uint32_t by, uint32_t bz, const YieldCtl ctl) {
    run_tile<true>(a, bx, by, bz, ctl);
  }
  // (YIELD: the best-effort form, which covers blocks of 256 rows and 128 columns and writes past the caches)
  template <bool YIELD>
  static __device__ __forceinline__ void run_tile(const Args &a, uint32_t bx, uint32_t by, uint32_t bz, const YieldCtl ctl) {
#ifdef __HIP_DEVICE_COMPILE__
    extern __shared__ __align__(1024) unsigned char tally_dyn_lds[];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wm = wave >> 1, wn = wave & 1;
    const uint32_t K = a.k;
    const uint32_t LDA = a.lda ? a.lda : K, LDB = a.ldb ? a.ldb : K;
    const uint32_t ns = (K + 63) / 64;
    // A load moves 8 rows x 128 bytes to 1 KB of LDS; lane l supplies 16-byte slot l, that is row l/8, k-chunk
    // (l%8) xor ((row/2)%8).  Load j of a wave takes rows 8 (4 j + wave) on.  A lane whose offset has its top bit
    // set is outside the buffer and its slot is filled with zeros: rows past the matrix, k past K in a last stage
    // that is half full.
    constexpr uint32_t OOB = 0x80000000u;
    const buf_t rA = make_buf(a.A + bz * a.stride_a + (uint64_t)by * TM * LDA, 0x7fffffffu);
    const buf_t rB = make_buf(a.Bt + bz * a.stride_b + (uint64_t)bx * TN * LDB, 0x7fffffffu);
    const uint32_t r8 = lane >> 3, c8 = (lane & 7) ^ (lane >> 4) ^ ((wave & 1) * 4);
    uint32_t v[L];                                         // A's, then B's
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const bool isA = j < RA;
      const uint32_t r = ((isA ? j : j - RA) * 4 + wave) * 8 + r8;
      v[j] = (isA ? by * TM + r < a.m : bx * TN + r < a.n) ? (r * (isA ? LDA : LDB) + c8 * 8) * 2 : OOB;
    }
    const uint32_t base = (uint32_t)(uintptr_t)(lptr_t)tally_dyn_lds, end = base + R * STAGE;
    uint32_t to = base + wave * 1024, so = 0, left = ns;   // the next stage to ask for: its place, its k in bytes, how many
    auto open = [&]() {                                    // before a stage's loads
      if (--left == 0 && (K & 32)) {
        const uint32_t none = c8 & 4 ? OOB : 0u;
#pragma unroll
        for (int j = 0; j < L; ++j) v[j] |= none;
      }
    };
    auto load = [&](int j) {
      const uint32_t at = to + (j < RA ? j * 4096 : SA + (j - RA) * 4096);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(j < RA ? rA : rB, (lptr_t)at, 16, v[j], so, 0, 0);
    };
    auto close = [&]() {
      so += 128;
      to = to + STAGE >= end ? to + STAGE - R * STAGE : to + STAGE;
    };
    // lane l takes row l%16 of a 16-row block, k-chunk 4 kk + l/16; two sets, this stage's and the next one's
    const uint32_t f_off = (lane & 15) * 128 + (((lane >> 4) ^ ((lane >> 1) & 7)) * 16);
    const uint32_t fA = wm * (16 * RA * 128) + f_off, fB = SA + wn * (16 * RB * 128) + f_off;
    typedef const volatile __attribute__((address_space(3))) bf16x8_t *frag_t;   // (volatile: pinned)
    bf16x8_t fa[2][2][RA], fb[2][2][RB];
    uint32_t from = base;                                  // place of the next stage to read
    auto read = [&](int f, int i) {                        // the i-th of 2 L
      const int kk = i / L, j = i % L;
      if (j < RB) fb[f][kk][j] = *(frag_t)(from + (fB ^ (kk * 64)) + j * 2048);
      else fa[f][kk][j - RB] = *(frag_t)(from + (fA ^ (kk * 64)) + (j - RB) * 2048);
    };
    auto advance = [&]() { from = from + STAGE == end ? base : from + STAGE; };
    f32x4_t acc[RA][RB];
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
      for (int j = 0; j < RB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // A stage whose fragments are in registers or on their way there: once everybody's are, its place is free, and
    // once no more than AFTER stages are on their way the next one has landed.  Behind each MFMA goes a share of the
    // next stage's reads and of the loads into the place that became free.
    auto step = [&](auto after, auto set, auto next, auto more) {
      constexpr int AFTER = decltype(after)::value, f = decltype(set)::value;
      constexpr bool READ = decltype(next)::value, LOAD = decltype(more)::value;
      if constexpr (READ) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L * AFTER) : "memory");
      __builtin_amdgcn_s_waitcnt(0xc07f);                  // lgkmcnt(0)
      if constexpr (READ) __builtin_amdgcn_s_barrier();
      if constexpr (LOAD) open();
      __builtin_amdgcn_sched_barrier(0);
      constexpr int M = 2 * RA * RB, O = 3 * L;
#pragma unroll
      for (int q = 0; q < M; ++q) {
        const int kk = q / (RA * RB), i = q % (RA * RB) / RB, j = q % RB;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[f][kk][j], fa[f][kk][i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = q * O / M; o < (q + 1) * O / M; ++o) {
          if (o % 3 != 2 && READ) read(f ^ 1, o / 3 * 2 + o % 3);
          if (o % 3 == 2 && LOAD) load(o / 3);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (READ) advance();
      if constexpr (LOAD) close();
    };
    typedef std::integral_constant<int, 0> set0;
    typedef std::integral_constant<int, 1> set1;
    typedef std::integral_constant<int, R - 2> full;
    auto pair = [&]() {
      step(full{}, set0{}, std::true_type{}, std::true_type{});
      step(full{}, set1{}, std::true_type{}, std::true_type{});
    };
    auto to_set0 = [&]() {                                 // the fragments just read
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int i = 0; i < RA; ++i) fa[0][kk][i] = fa[1][kk][i];
#pragma unroll
        for (int j = 0; j < RB; ++j) fb[0][kk][j] = fb[1][kk][j];
      }
    };
    auto begin = [&]() {
#pragma unroll
      for (int i = 0; i < 2 * L; ++i) read(0, i);
      advance();
    };
    auto request = [&]() {
      open();
#pragma unroll
      for (int j = 0; j < L; ++j) load(j);
      close();
    };
    // Looks at the pause word (see GemmTileT): one lane asks among the operands' loads at the start of a round and
    // has the answer at the start of the next; the last question goes out before the last R stages.
    uint32_t pause_left = ctl.ticks, look = 0;
    const buf_t rF = make_buf(ctl.flag, YIELD && ctl.ticks != 0 ? 4 : 0);
    const uint32_t v_look = threadIdx.x == 0 ? 0u : OOB, look_mask = (ctl.mask >> 1) & ~(ROUND - 1u);   // in stages
    auto act = [&]() {
      if (YIELD && __builtin_amdgcn_readfirstlane(look) == ctl.epoch) yield_while_preempted(ctl, pause_left);
    };
    auto look_round = [&](bool ask) {
      act();
      look = __builtin_amdgcn_raw_buffer_load_b32(rF, v_look | (ask ? 0u : OOB), 0, 16);  // (sc1)
    };
    // the last stages, AFTER of them behind this one: nothing is asked for any more
    auto finish = [&](auto &&self, auto after, auto set) -> void {
      constexpr int AFTER = decltype(after)::value, f = decltype(set)::value;
      if constexpr (YIELD && AFTER == 1) {
        static_assert(R - 2 <= ROUND || !YIELD, "an answer is acted on a round later");
        act();
      }
      step(std::integral_constant<int, (AFTER > 0 ? AFTER - 1 : 0)>{}, set, std::bool_constant<(AFTER > 0)>{}, std::false_type{});
      if constexpr (AFTER > 0) self(self, std::integral_constant<int, AFTER - 1>{}, std::integral_constant<int, f ^ 1>{});
    };
    if constexpr (YIELD) {
      if (ctl.look_first && ctl.ticks != 0 && wave == 0 && ns >= 16) yield_while_preempted(ctl, pause_left);
      __syncthreads();                                     // (LDS may have been another tile's)
    }
    if (ns >= (uint32_t)R) {
#pragma unroll
      for (int d = 0; d < R; ++d) request();
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L * (R - 1)) : "memory");
      __builtin_amdgcn_s_barrier();
      begin();
      uint32_t c = ns - R;
      if (c & 1) {
        step(full{}, set0{}, std::true_type{}, std::true_type{});
        __builtin_amdgcn_s_waitcnt(0xc07f);
        to_set0();
      }
      c >>= 1;
      if constexpr (YIELD) {
        if (ROUND == 4) {
          if (c & 1) pair();
          c >>= 1;
        }
        for (; c; --c) {
          look_round((c * ROUND & look_mask) == look_mask);
          pair();
          if (ROUND == 4) pair();
        }
        look_round(true);
      } else {
        for (; c; --c) pair();
      }
      finish(finish, std::integral_constant<int, R - 1>{}, set0{});
    } else {
      for (uint32_t d = 0; d < ns; ++d) request();
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      begin();
      for (uint32_t d = 1; d < ns; ++d) {
        step(set0{}, set0{}, std::true_type{}, std::false_type{});
        __builtin_amdgcn_s_waitcnt(0xc07f);
        to_set0();
      }
      step(set0{}, set0{}, std::false_type{}, std::false_type{});
    }
#pragma unroll
    for (int i = 0; i < RA; ++i)
      store_blocks<NAN7FC0, YIELD>(a, bz, by * TM + (wm * RA + i) * 16 + (lane & 15), bx * TN + wn * 16 * RB, lane, acc[i]);
#endif
  }
};
// The small GEMM's own blocks stop at their ends only, as its waves fit beside a request's.
struct GemmSmallBody : GemmTileT<1, 1, true> {
  static constexpr bool TEAMS = true;
  static uint64_t block_bytes(const Args &a) { return 128 * (uint64_t)a.k; }
  // (us and us of drain with the counter alone / in teams, 4096 x 4096: k = 512, 512 x 1 211 11.9 / 133 8.4; k = 384,
  // 256 x 1 205 7.6 / 191 7.5; of 2048 x 2048 in us, k = 1024, 256 x 1 64.9 / 69.9)
  static uint32_t team_bytes(uint32_t workers, uint32_t) { return workers >= 512 ? 64 << 10 : 48 << 10; }
  static constexpr bool YIELDS = false;
};

// Measured ceiling of the matrix pipe: every wave issues independent 32x32x16 bf16 MFMAs on
// register operands only (no LDS, no memory), one wave per SIMD on every compute unit, as
// a GEMM tile does.  The shader clock is power-managed, so the rate depends on how many
// units are busy and on the operand bits (random bits toggle more than zeros).
__global__ __launch_bounds__(256) void mfma_ceiling_kernel(const uint4 *operands, float *sink,
                                                           uint32_t iters) {
  const uint4 va = operands[threadIdx.x & 63], vb = operands[64 + (threadIdx.x & 63)];
  const bf16x8_t fa = __builtin_bit_cast(bf16x8_t, va), fb = __builtin_bit_cast(bf16x8_t, vb);
  f32x16_t acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  for (uint32_t it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc[i], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += acc[i][r];
  sink[blockIdx.x * 256 + threadIdx.x] = s;
}

}  // namespace tally
