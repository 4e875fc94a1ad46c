// Which tiles cover the output of a GEMM in its original form, and which of them a workgroup takes.  Plain C++
// beside the kernels: the rules can be looked at without a GPU.
#pragma once
#include <stdint.h>

#include "../../include/tally.h"

#if defined(__HIPCC__)
#define TALLY_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define TALLY_HOST_DEVICE inline
#endif

namespace tally {

constexpr uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// bytes of output from which GemmBodyT writes it past the caches
constexpr uint64_t kGemmBigOutput = 128ull << 20;

// How an original form is launched: on the high-priority stream; beside best-effort workgroups that leave
// little LDS; beside any best-effort job.
constexpr uint32_t kUrgent = 1u, kBeside = 2u, kShared = 4u;

// How the original form of a GEMM covers its output: with the largest tiles that still leave no
// compute unit idle, whatever the logical blocks are (only slices and workers have to keep to
// those; the bits are the same, see GemmTileT).  Counted in tiles for 256 compute units; us at
// m x n x 2048 for 32x32 / 32x64 / 64x64 / 128x64 / 256x128 / 256x256 tiles:
//    512 x 512    6.6 /  8.5 / 11.6 / 17.0 / 24.6 / 40.4   (256 of 32x32)
//    512 x 768    9.8 /  8.7 / 11.7 / 17.1 / 24.6 / 40.5   (192 of 32x64)
//    512 x 1024  10.4 /  9.0 / 11.9 / 17.2 / 24.4 / 40.7   (256 of 32x64)
//    768 x 1024  13.9 / 13.5 / 12.2 / 17.3 / 24.4 / 40.6   (192 of 64x64)
//   1024 x 1024  17.4 / 14.4 / 12.8 / 17.8 / 25.2 / 40.9   (256; at k = 8192 56 / 43 / 41)
//   1024 x 2048  30.5 / 24.6 / 18.5 / 18.7 / 25.6 / 40.6   (512; 256 of 128x64)
//   2048 x 2048  53.9 / 42.1 / 31.2 / 26.2 / 26.3 / 40.8   (128 of 256x128)
//   2048 x 4096   106 / 71.5 / 51.7 / 43.6 / 30.2 / 42.1   (256 of 256x128)
//   4096 x 4096   192 /  135 / 98.0 / 83.3 / 58.0 / 51.9   (256 of 256x256)
// and the same order from k = 512 to 8192.  Below k = 128 there is no loop to speak of and the
// large tiles' long prologue and epilogue lose to 128x64 (4352 x 4864 x 64: 15.4 against 13.3),
// unless the output is one that GemmBodyT writes past the caches.
// Tiles of one wave (GemmWaveT) pay from the third stage on and where there are few of them: they keep more
// bytes on their way and fewer instructions between them, but read operands more often.  Counted in 16x16
// blocks of the output, us for 32x32 or 32x64 tiles, the better / 16x16 / 16x32 or 32x16 / the best GemmRingT,
// with both operands from the caches and from memory:
//  8192 x   16 x 1536 (512)    5.2 / 3.9 / 4.6 / 4.7     6.7 /  6.5 /  8.3 /  6.6
//    94 x  799 x 2464 (300)    6.8 / 5.3 / 6.2 / 6.1     7.3 /  5.5 /  7.2 /  6.5
//  1000 x  128 x 4096 (504)   10.1 / 7.3 / 9.1 / 8.6    11.6 / 10.0 / 14.5 / 10.7
//   512 x  384 x 1536 (768)    5.3 / 5.0 / 4.8 / 4.7     5.5 /  5.4 /  5.4 /  4.8
//   512 x  384 x 4096 (768)   10.3 / 9.1 / 9.3 / 8.8    11.1 / 13.6 / 15.0 / 10.4
//   256 x  768 x  928 (768)    4.1 / 3.5 / 3.8 / 3.8     4.3 /  3.8 /  4.1 /  3.9
//   200 x 1000 x  768 (819)    3.8 / 3.9 / 3.5 / 3.5     3.9 /  3.8 /  3.8 /  3.6
//  1000 x  256 x  320 (1008)   3.1 / 3.1 / 2.6 / 3.1     3.4 /  3.2 /  2.9 /  3.2
//    90 x 3400 x  768 (1278)   4.7 / 4.6 / 4.1 / 4.1     5.2 /  5.5 /  5.5 /  4.9
//   128 x 3072 x  768 (1536)   4.7 / 4.5 / 3.8 / 4.1     4.8 /  5.0 /  4.4 /  4.4
//  4096 x   96 x 1536 (1536)   7.1 / 7.4 / 6.2 / 5.8     7.6 / 11.3 /  9.6 /  7.4
//  2048 x  256 x  320 (2048)   3.4 / 4.6 / 3.1 / 3.4     3.7 /  4.9 /  3.2 /  3.6
//  2048 x  256 x  768 (2048)   4.7 / 5.8 / 4.3 / 4.3     4.9 /  6.2 /  4.5 /  4.3
// So 16x16 up to five for two compute units, or three for one up to k = 1024; then two blocks to a tile up to eight
// per unit, for k from three stages to eight, with the pair along the longer side only where the blocks of the
// shorter one are odd in number and a last tile would be half empty.  Of 473 products of up to 2048 blocks, more tall than wide, two
// take over 4 % longer than in tiles through registers (16384 x 32 x 4096 from memory, 33.4 and 31.9); the mean is
// 0.83 of those with operands from the caches and 0.87 from memory, 0.88 and 0.90 beside best-effort jobs.
// Beside best-effort workgroups that leave LDS for one of them on a compute unit (kBeside) more than 256 would
// run in rounds: there operands go through registers (the nine-kernel layer beside paused 256x256 tiles 43.5 us
// from the request to its completion, 54 in one-wave tiles throughout).
// Where nobody else needs the LDS (kShared is not set) GemmRingT covers everything that is less than 160 tiles of
// 256x256, from k = 320 on, k = 160 up to 2048 blocks of 16x16, or k = 128 where there are more than 512 tiles of
// 64x64.  The tile is the one for which the model at GemmRingT says the least: (RA + RB) for each stage of as many
// tiles as a compute unit gets, and 10 + 8 (RA + RB) of those units, of 0.05 us, for every time it starts anew.  One tile
// after the other on a unit that holds one at a time is a fifth slower than that (3000 x 3000 x 2048 in 128x96
// 48.6 us, 42.7 in 96x96, two on a unit); five stages ahead instead of three are a tenth faster and 1 us longer under
// way (1280 x 1280 x 4096 22.2 and 19.9, x 768 6.0 and 6.6); 256x128 tiles count as 16.5 (17.8 in a batch, whose
// tiles are not dealt out to the dies by product), 256x256 tiles as 20.5 and 24 x 10 to start, 128x64 through
// registers as 7.8, four on a unit (2048 x 4096 x 448 in those 13.8 us, 15.2 in 128x128 or 96x96).
// Without the large tiles among them, where smaller ones need another round for a few: us in the best of the others
// / 256x256: 3 of 5632 x 512 x 768 36.2 (128x64) / 20.4, 3 of 1280 x 2560 x 2400 66.9 / 51.9,
// 3328 x 3072 x 6304 153 (128x128) / 111.  Of 597 products of k = 128 to 8192 the choice takes 1 % longer than the
// best tile in the mean, and over 6 % longer in 49 with operands from the caches and 29 from memory.
// For less work tiles through registers are as fast or faster (1024 x 1024 x 256 3.64 us, 3.78 in 64x64).
// None of them fills more of a compute unit than 128 KB alone or 160 KB as two that come and go: beside the long ones,
// which may be a best-effort product's, a request's tiles through registers find 16 to 24 KB (1280 x 1280 x 4096 in
// tiles of 144 KB, 128 x 768 x 3072 beside it 30.7 us from the call to its end, 21.6 so).
enum class GemmCover { k32, k32x64, k64, k128x64, k256x128, k256x256, kWave16, kWave16x32, kWave32x16, kRing };
#define GEMM_RINGS(X) X(1, 1, 8) X(1, 2, 6) X(2, 2, 5) X(2, 3, 4) X(4, 2, 3) X(3, 3, 3) X(4, 2, 5) X(3, 3, 5) X(4, 3, 4) X(4, 4, 4)
constexpr uint32_t ring_per_cu(uint32_t ra, uint32_t rb, uint32_t r) { return 160 * 1024 / (32 * (ra + rb) * 128 * r); }
#define GEMM_RING_ROW(ra, rb, r) {32 * ra, 32 * rb, ring_per_cu(ra, rb, r), r},
constexpr uint32_t kRings[][4] = {GEMM_RINGS(GEMM_RING_ROW)};   // tile, how many fit a compute unit, stages
constexpr uint32_t kRingCount = sizeof(kRings) / sizeof(kRings[0]);
// large: the columns of the operator's blocks of 256 rows (0: it has none)
inline GemmCover gemm_ring(const tally_gemm_bf16_args &a, uint32_t large) {
  const uint64_t ns = cdiv(a.k, 64);
  const uint64_t through = (uint64_t)cdiv(a.m, 128) * cdiv(a.n, 64) * a.batch;   // 128x64 tiles through registers
  GemmCover best = GemmCover::k128x64;
  uint64_t least = cdiv(through, 256) * ns * 78 + cdiv(through, 1024) * 880;
  for (uint32_t tn = 128; tn <= large; tn += 128) {
    const uint64_t rounds = cdiv((uint64_t)cdiv(a.m, 256) * cdiv(a.n, tn) * a.batch, 256);
    const uint64_t cost = rounds * (tn == 128 ? (a.batch == 1 ? 165 : 178) * ns + 1060 : 205 * ns + 1200);
    if (cost < least) {
      least = cost;
      best = tn == 128 ? GemmCover::k256x128 : GemmCover::k256x256;
    }
  }
  for (uint32_t i = 0; i < kRingCount; ++i) {
    const uint64_t t = (uint64_t)cdiv(a.m, kRings[i][0]) * cdiv(a.n, kRings[i][1]) * a.batch, rounds = cdiv(t, 256);
    const uint64_t size = (kRings[i][0] + kRings[i][1]) / 32, per_cu = kRings[i][2];
    const bool deep = per_cu == 1 && kRings[i][3] >= 5;
    const uint64_t unit = per_cu == 1 && rounds > 1 ? 24 : deep ? 17 : 20;   // half units
    const uint64_t cost = rounds * ns * size * unit / 2 + cdiv(t, 256 * per_cu) * 10 * (10 + 8 * size + (deep ? 20 : 0));
    if (cost < least) {
      least = cost;
      best = (GemmCover)((uint32_t)GemmCover::kRing + i);
    }
  }
  return best;
}
// large: as above; such blocks cover the output without a remainder
inline GemmCover gemm_cover(const tally_gemm_bf16_args &a, uint32_t how, uint32_t large) {
  const uint64_t t16 = (uint64_t)cdiv(a.n, 16) * cdiv(a.m, 16) * a.batch, t64 = (uint64_t)cdiv(a.n, 64) * cdiv(a.m, 64) * a.batch;
  const bool ring = !(how & kShared) && t64 <= (1u << 20) &&         // (a flat grid)
                   a.k >= (t64 > 512 ? 128u : t16 <= 2048 ? 160u : 320u);
  if (a.k > 128 && (!(how & kBeside) || t16 <= 256)) {
    if (t16 <= (a.k <= 1024 ? 768u : 640u)) return GemmCover::kWave16;
    if (t16 <= 2048 && a.k > 160 && a.k <= 512) {
      const bool tall = a.m > a.n, odd = cdiv(tall ? a.n : a.m, 16) & 1;   // (the shorter side)
      return tall != odd ? GemmCover::kWave16x32 : GemmCover::kWave32x16;
    }
  }
  if (ring && !(large && (uint64_t)cdiv(a.n, 256) * cdiv(a.m, 256) * a.batch >= 160)) return gemm_ring(a, large);
  if ((uint64_t)cdiv(a.n, 32) * cdiv(a.m, 32) * a.batch <= 256) return GemmCover::k32;
  if ((uint64_t)cdiv(a.n, 64) * cdiv(a.m, 32) * a.batch <= 256) return GemmCover::k32x64;
  if (t64 <= 512) return GemmCover::k64;
  if (a.k <= 128 && (uint64_t)a.m * a.n * a.batch * 2u <= kGemmBigOutput) return GemmCover::k128x64;
  if ((uint64_t)cdiv(a.n, 128) * cdiv(a.m, 256) * a.batch <= 256) return GemmCover::k256x128;
  return GemmCover::k256x256;
}
// The ragged GEMM: only the tiles with predicated edges, which also fit beside a paused
// best-effort tile.  128x64 tiles pay from two per compute unit (512 x 4096 x 4096, 256 of them,
// 29 us with 64x64 and 32; 1024 x 4096 x 4096, 512, 54 and 47).
inline GemmCover gemm_cover_small(const tally_gemm_bf16_args &a, uint32_t how) {
  const GemmCover c = gemm_cover(a, how, 0);
  if (c <= GemmCover::k32x64 || c >= GemmCover::kWave16) return c;
  return (uint64_t)cdiv(a.n, 64) * cdiv(a.m, 128) * a.batch >= 512 ? GemmCover::k128x64 : GemmCover::k64;
}
// Workgroup (die, in, at) of GemmWaveT: the panel `at` of the die's run of them, tile `in` of the panel (see there).
TALLY_HOST_DEVICE bool wave_tile(const tally_gemm_bf16_args &a, uint32_t tm, uint32_t tn, uint32_t die, uint32_t in, uint32_t at,
                                 uint32_t *bx, uint32_t *by, uint32_t *bz) {
  const bool tall = a.m > a.n;
  const uint32_t panels = tall ? (a.m + tm - 1) / tm : (a.n + tn - 1) / tn;   // of a product
  const uint32_t q = panels * a.batch / 8, rest = panels * a.batch % 8;
  if (at >= q + (die < rest ? 1 : 0)) return false;
  uint32_t panel = die * q + (die < rest ? die : rest) + at;
  *bz = 0;
  if (a.batch > 1) {
    *bz = panel / panels;
    panel -= *bz * panels;
  }
  *bx = tall ? in : panel;
  *by = tall ? panel : in;
  return true;
}

// Workgroup `id` of GemmRingT's flat grid (see there).
TALLY_HOST_DEVICE bool ring_tile(const tally_gemm_bf16_args &a, uint32_t tm, uint32_t tn, uint32_t id, uint32_t *bx, uint32_t *by,
                                 uint32_t *bz) {
  const uint32_t X = (a.n + tn - 1) / tn, Y = (a.m + tm - 1) / tm, T = X * Y * a.batch, q = T / 8, rest = T % 8;
  const uint32_t die = id & 7, at = id >> 3;
  if (at >= q + (die < rest ? 1 : 0)) return false;
  uint32_t t = die * q + (die < rest ? die : rest) + at;
  *bz = t / (X * Y);
  t -= *bz * (X * Y);
  const uint32_t H = q >= 48 ? 8 : q >= 12 ? 4 : 2;
  const uint32_t band = t / (H * X), in = t - band * H * X, h = Y - band * H < H ? Y - band * H : H;
  *bx = in / h;
  *by = band * H + (in - *bx * h);
  return true;
}

}  // namespace tally
