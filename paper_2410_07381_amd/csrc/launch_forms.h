// The three launch forms of a best-effort kernel, generated from one logical-block body.
//
// A Body is a struct with
//   using Args = <POD passed by value to the kernel>;
//   static constexpr int THREADS;            threads per logical block
//   static constexpr int MIN_WAVES;          waves per SIMD the compiler must leave room for
//   static constexpr unsigned DYN_LDS;       dynamic LDS bytes the body needs
//   static constexpr bool END_BARRIER;       true if consecutive blocks run by one workgroup
//                                            would race on workgroup-shared state
//   static constexpr bool YIELDS;            true if the body offers run_yielding(), which
//                                            pauses inside the block while preempted
//   static constexpr bool RANGE;             true if the body offers run_range(args, first,
//                                            last) for consecutive blocks of a 1-D grid
//   static __device__ void run(const Args&, uint32_t bx, uint32_t by, uint32_t bz);
//   static __device__ void run_be(const Args&, uint32_t bx, uint32_t by, uint32_t bz);
// run() performs the work of original block (bx,by,bz); run_be() is the same work as the
// best-effort forms (sliced, persistent workers) do it: identical arithmetic (a kernel's outputs
// are the same bits in every form, wherever a job was stopped), but data that
// is touched once goes through non-temporal accesses so that it does not evict the
// high-priority job's data from the caches; every thread of the workgroup
// calls it and returns from it (no early exit), so the workgroup-wide barriers of the
// persistent-worker loop are reached by all threads (Section 4.1: divergent barriers
// stall a kernel for ever; hand-written bodies handle ragged tails by predication).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/tally.h"

namespace tally {

// A preemption request is folded into the task counter by adding this to it: every later
// fetch then returns an index beyond any grid (grids have fewer than 2^30 blocks).
constexpr uint32_t kPreemptStep = 0x80000000u;
// Bit of the host's request word that says "do not pause inside blocks".
constexpr uint32_t kNoPauseBit = 0x80000000u;

// Coverage record of a logical block on the device.  `block.count` counts executions of it as a
// whole; one handed out in P parts adds 64 / P pieces per part, and to `which` the bits of the
// pieces.  All of them were run once exactly where 64 pieces add up to 64 one bits: no other 64
// powers of two below 2^64 have that sum, whatever carries (tally_parts_executions).
struct CoverRec {
  tally_cover_rec block;
  uint32_t pieces;
  unsigned long long which;
};
constexpr uint32_t kCoverPieces = 64;

// Workers in teams.  One word takes a fetch-and-add every 11.4 ns whoever asks (in any kind of
// memory): 256 workers on short blocks get one every 2.9 us, 512 every 5.8, and queue at the task
// counter for most of their time.  Words of their own serve eight workers each in 0.4 us: a
// team draws kTeamBatch fetches at once from the task counter and gives them out from its word,
// whose high half is what the counter held and whose low half counts the fetches given out.
// Whoever finds the batch used up first draws the next one, the others ask again until it is there.
//
// To the protocol a batch is a fetch: it is drawn by one fetch-and-add whose result says whether a
// request stands, and its indices are given out in order and run whatever happens next.  A worker
// leaves when its team's word gives it an index beyond the end, so nothing drawn is left behind (in
// a single pass, where each worker takes one, teams are whole batches).  The drawer waits for
// nothing, so neither do the others for long: while a draw is under way the count is beyond
// kTeamBatch, and nobody else gets the count that means "draw".  After a request the
// workers of a team finish what they hold and what is left of the batch, up to seven fetches among
// them: mostly one each, but whoever is free takes the next, so one worker may run all of them while
// the others are held up.
// Leaving is counted by teams too; a team's last worker puts its line back.
//
// Batches twice the team kept half of it waiting (SAXPY of 2^20, 256 x 1: 47 us against 30, and 54
// without teams); teams of four: 29, but 766 where teams of eight take 440 (2^26, 1024 x 1; 3002
// without).  Teams of neighbours, whose fetches go to all dies as they would without teams, beat
// those of one die by up to 9 % (LayerNorm of 300000 x 200, 512 x 1: 315 and 345 us, 866 without).
struct alignas(128) TeamLine {
  unsigned long long word;
  uint32_t left;
};
constexpr uint32_t kTeamBatch = 8, kTeamSize = 8, kMaxTeams = 256;
constexpr unsigned long long kTeamIdle = kTeamBatch;       // used up: the first to ask draws

// Device-side control block of one persistent-worker launch segment.
struct PtbCtl {
  uint32_t *counter;        // device: THE shared word.  Next task index (+ counter_base), plus
                            // kPreemptStep once a preemption request has been folded in.  It is
                            // never reset and wraps; indices are differences modulo 2^32.
  uint32_t *exited;         // device: workers (or teams) that have exited, summed over all segments
  unsigned long long *pre;  // device: (epoch << 32 | progress) written by the relay right after
                            // it folded a request in: what its fetch-and-add returned
  const uint32_t *host_flag;  // pinned host memory: epoch the host wants preempted (| kNoPauseBit)
  unsigned long long *host_status;  // pinned: (epoch << 32 | progress) once drained
  uint32_t *host_live;      // pinned: progress mirrored while running
  unsigned long long *host_raw;     // pinned: (epoch << 32 | raw counter) at the drain
  unsigned long long *host_relay;   // pinned: (epoch << 32 | raw counter) when the relay has ended
  unsigned long long *host_gave_up; // pinned: (epoch << 32 | 1 if the relay gave up early), written with it
  CoverRec *cover;          // device, may be null
  uint32_t parts;           // the counter counts parts of a logical block (1: whole blocks)
  uint32_t limit;           // workers treat this as the end of the grid (normally all of it); in parts
  uint32_t last_from;       // task indices from here on stand for fewer blocks a fetch (see block_at; none: `limit`)
  uint32_t last_chunk;      // blocks of such a fetch
  uint32_t end;             // the end of the grid in blocks (in parts where blocks have several)
  uint32_t epoch;           // id of this launch segment, unique for the life of the slot
  uint32_t exit_target;     // value of *exited after the last worker (or team) of this segment leaves
  uint32_t counter_base;    // raw counter value that stands for task index 0 of this job
  uint32_t workers;
  uint32_t chunk;           // task indices per fetch (1 where blocks have several parts)
  uint32_t single_pass;     // the workers' first fetches cover every index left: none fetches twice
  uint32_t whole;           // fetches of whole blocks per worker before it takes parts (TailBody)
  uint32_t segment;         // 0-based segment number, for the coverage records
  uint32_t gx, gy;          // logical grid extents (x fastest)
  uint32_t yield_ticks;     // longest pause inside ONE block, in 10 ns wall-clock ticks (0: never)
  uint32_t yield_mask;      // a pausing body looks at the pause word every (yield_mask + 1) steps
  uint32_t *flag_copies;    // device: kFlagCopies copies of the pause request (the epoch while
                            // workers are to pause inside their blocks, else 0), 128 B apart, for
                            // the mid-block polls (one address serves only ~80 M coherent scalar
                            // loads per second, whoever asks)
  TeamLine *teams;          // device: the slot's lines, one per team (`team_count` in use)
  uint32_t team_count;      // 0: every worker fetches and leaves by itself
};
constexpr uint32_t kFlagCopies = 64;
constexpr uint32_t kFlagCopyStride = 32;  // in 32-bit words

// The last round of fetches, shared.  A grid of B blocks taken C at a time by W workers ends with a
// round in which only B mod (W C) blocks are left: as whole fetches they keep a few workers busy for as
// long as a full round, so in that round a fetch brings as many blocks as give every worker one
// (`last_chunk`).  A fetch still advances the counter by `chunk`; from `last_from` on, `chunk` task
// indices stand for `last_chunk` blocks.  Nothing else knows: an index is turned into blocks where a
// worker runs it and where progress is told to the host.
// Softmax as 256 x 4, whole fetches / so, us: 9001 x 8192 (51 third fetches / 203 of one block) 142 / 126,
// 700 x 6000 (44 fetches / 175) 39 / 23, 5000 x 2048 32.8 / 29.6 (see last_round).
__device__ __forceinline__ uint32_t block_at(const PtbCtl &c, uint32_t index) {
  if (index <= c.last_from) return index;
  const uint32_t b = c.last_from + (index - c.last_from) / c.chunk * c.last_chunk;
  return b < c.end ? b : c.end;
}

struct SliceCtl {
  CoverRec *cover;
  uint32_t offset;          // first logical block of this sub-kernel
  uint32_t gx, gy;
  uint32_t segment;
};

__device__ __forceinline__ void delinearize(uint32_t idx, uint32_t gx, uint32_t gy, uint32_t &bx,
                                            uint32_t &by, uint32_t &bz) {
  bx = idx % gx;
  uint32_t r = idx / gx;
  by = r % gy;
  bz = r / gy;
}

__device__ __forceinline__ void record_at(tally_cover_rec &r, uint32_t bx, uint32_t by, uint32_t bz,
                                          uint32_t segment, uint32_t worker) {
  r.bx = bx; r.by = by; r.bz = bz; r.segment = segment; r.worker = worker;
}
__device__ __forceinline__ void record(CoverRec *cover, uint32_t idx, uint32_t bx, uint32_t by, uint32_t bz,
                                       uint32_t segment, uint32_t worker) {
  if (cover != nullptr && threadIdx.x == 0) {
    atomicAdd(&cover[idx].block.count, 1u);
    record_at(cover[idx].block, bx, by, bz, segment, worker);
  }
}
// part `part` of `parts` (at least 2) of block idx; block index, segment and worker are the first part's
__device__ __forceinline__ void record_part(CoverRec *cover, uint32_t idx, uint32_t part, uint32_t parts, uint32_t bx,
                                            uint32_t by, uint32_t bz, uint32_t segment, uint32_t worker) {
  if (cover != nullptr && threadIdx.x == 0) {
    const uint32_t w = kCoverPieces / parts;
    atomicAdd(&cover[idx].pieces, w);
    atomicAdd(&cover[idx].which, ((1ull << w) - 1) << (part * w));
    if (part == 0) record_at(cover[idx].block, bx, by, bz, segment, worker);
  }
}

// ---- original form -------------------------------------------------------------------
// `urgent` marks a launch on the high-priority stream: its waves raise their own issue
// priority so that, where they share a SIMD with a best-effort wave that is still
// finishing its block, the arbiter picks their instructions first.
template <class Body>
__global__ __launch_bounds__(Body::THREADS, Body::MIN_WAVES) void native_kernel(typename Body::Args args,
                                                               uint32_t urgent) {
  if (urgent) __builtin_amdgcn_s_setprio(3);
  Body::run(args, blockIdx.x, blockIdx.y, blockIdx.z);
}



// ---- sliced form: logical block = offset + blockIdx (Section 4.1, slicing) -----------
template <class Body>
__device__ __forceinline__ void sliced_body(const typename Body::Args &args, const SliceCtl &ctl) {
  uint32_t idx = ctl.offset + blockIdx.x, bx, by, bz;
  delinearize(idx, ctl.gx, ctl.gy, bx, by, bz);
  Body::run_be(args, bx, by, bz);
  record(ctl.cover, idx, bx, by, bz, ctl.segment, blockIdx.x);
}
template <class Body>
__global__ __launch_bounds__(Body::THREADS, Body::MIN_WAVES) void sliced_kernel(typename Body::Args args,
                                                               SliceCtl ctl) {
  sliced_body<Body>(args, ctl);
}

// ---- persistent-worker form (Section 4.1, preemption) --------------------------------
// The paper's worker reads a flag, then fetches and increments the task counter: two
// dependent round trips to memory per iteration.  Here the flag lives in the counter: a
// request is raised by adding 2^31 to it, a worker does ONE fetch-and-add per iteration
// and leaves when the index it got is beyond the grid, whether the grid is exhausted or a
// request was folded in.  A fetched index is always run (check and fetch are one
// operation, so the order question does not arise).
//
// The host raises a request with one store to pinned host memory (cheap to write, but a
// load from it crosses PCIe, far too slow for hundreds of workers to poll).  A one-wave
// relay kernel, launched just before the workers on a stream of its own, polls that word;
// when it names this segment the relay folds the request into the counter (its
// fetch-and-add returns the exact progress, which it leaves in `pre` for the last worker
// to publish) and, unless the request says otherwise, raises the pause word that workers
// inside long blocks poll.  It mirrors the progress to the host and leaves when every
// worker of the segment has exited, so its lifetime is bounded by the workers', which
// depend on nothing.
//
// The relay polls with scalar loads that bypass the scalar cache: a vector load that
// waits a microsecond on PCIe sits in the compute unit's vector-memory return queue in
// front of the loads of whatever worker shares that unit (measured: that worker's GEMM
// tile ran 20 % longer, and with it the whole kernel); the scalar path is separate.
__device__ __forceinline__ uint32_t scalar_load_coherent(const uint32_t *p) {
  uint32_t v;
  asm volatile("s_load_dword %0, %1, 0x0 glc\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(p) : "memory");
  return v;
}

constexpr unsigned long long kRelayGiveUpTicks = 2000000ull;  // 20 ms of the 100 MHz clock

__global__ __launch_bounds__(64) void relay_kernel(PtbCtl c) {
  uint32_t last = 0u;        // the host's word is 0 while nothing is asked
  bool added = false, gave_up = false;
  // The relay is launched before its workers.  Where the two cannot run side by side
  // (kernels executed strictly one after another) the workers cannot start until the
  // relay has ended: it leaves when neither the task counter nor the exit counter has
  // moved (by anyone but itself) for 20 ms; a request it folded in before that stands,
  // and the workers then find it when they start.
  const unsigned long long born = wall_clock64();
  uint32_t ctr0 = scalar_load_coherent(c.counter);
  const uint32_t gone0 = scalar_load_coherent(c.exited);
  bool alive = false;
  uint32_t mirrored = 0u;
  for (uint32_t n = 0;; ++n) {
    // once the request is in the counter only its withdrawal (the end of a pause) is news
    // from the host, and the exit counter is what matters: look at the host less often
    // (host's word and exit counter one after the other, about 2 us a round: asked for together
    // they made the worker beside the relay fall behind the others, 100 us of a training-like
    // step of 7890, and slower rounds are felt by the requests)
    uint32_t want = last;
    if (!added || (n & 3u) == 0u) want = scalar_load_coherent(c.host_flag);
    if (want != last) {
      const bool mine = (want & ~kNoPauseBit) == c.epoch;
      if (mine && !added) {
        uint32_t p = 0;
        if (threadIdx.x == 0) {
          const uint32_t old = __hip_atomic_fetch_add(c.counter, kPreemptStep, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
          p = old - c.counter_base;
          p = p < c.limit ? p : c.limit;
          __hip_atomic_store(c.pre, ((unsigned long long)c.epoch << 32) | p, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(c.host_live, block_at(c, p) / c.parts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        added = true;
        ctr0 += kPreemptStep;
      }
      // pause word: this segment's epoch while its workers are to pause inside blocks
      const uint32_t pause = (mine && !(want & kNoPauseBit)) ? c.epoch : 0u;
      if (c.flag_copies != nullptr && threadIdx.x < kFlagCopies)
        __hip_atomic_store(c.flag_copies + threadIdx.x * kFlagCopyStride, pause, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      last = want;
    }
    // the counters of a slot only ever grow (they are never reset), so a relay that
    // starts late, even after its workers are long gone, still sees the target passed
    uint32_t gone = scalar_load_coherent(c.exited);
    if ((n & 255u) == 255u)  // and, now and then, through the path the workers' atomics use
      gone = __hip_atomic_load(c.exited, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((int32_t)(gone - c.exit_target) >= 0) break;
    if ((n & 15u) == 0u) {
      const uint32_t raw = scalar_load_coherent(c.counter);
      if (raw != ctr0 || gone != gone0) alive = true;
      if (!alive && wall_clock64() - born > kRelayGiveUpTicks) { gave_up = true; break; }
      // (only news: a store to the host occupies the vector-memory queue of the compute unit for a
      // microsecond, and whichever worker shares that unit falls behind the others)
      const uint32_t ctr = raw - c.counter_base, live = block_at(c, ctr < c.limit ? ctr : c.limit) / c.parts;
      if (!added && live != mirrored) {
        if (threadIdx.x == 0)
          __hip_atomic_store(c.host_live, live, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        mirrored = live;
      }
    }
  }
  // Last act: tell the host that this relay will not touch the counter any more, and what
  // the counter holds now (every worker has exited unless the relay gave up, in which case
  // the last worker's own report is the final one).
  if (threadIdx.x == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no mirrored progress may land after this report)
    const uint32_t raw = __hip_atomic_load(c.counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // (each word carries the epoch: the host waits for both, so they need no order)
    const unsigned long long tag = (unsigned long long)c.epoch << 32;
    __hip_atomic_store(c.host_gave_up, tag | (gave_up ? 1u : 0u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(c.host_relay, tag | raw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Pause inside a long block while a preemption request stands.  Block-level preemption
// cannot act before the end of the running block; a block that lasts hundreds of
// microseconds (a 256x256 GEMM tile over a long K) would keep competing with the
// high-priority kernel for memory bandwidth and issue slots all that time.  Such a body
// calls this every few steps: the wave sleeps, holding its registers and LDS (the
// high-priority kernel runs beside it), until the request is withdrawn or the block's
// pause budget is spent, so a high-priority kernel that does NOT fit beside it cannot
// deadlock.  The budget is per block: `left` carries what remains of it across the polls.
struct YieldCtl {          // passed by value: taking the address of the kernel's control
  const uint32_t *flag;    // block would force it out of scalar registers into memory
  uint32_t epoch, ticks;
  uint32_t mask;           // poll when (step & mask) == mask
  bool look_first;         // the block may begin during a request: it does not follow a fetch at once
};
__device__ __forceinline__ void yield_while_preempted(const YieldCtl &y, uint32_t &left) {
  if (left == 0u || scalar_load_coherent(y.flag) != y.epoch) return;
  const unsigned long long t0 = wall_clock64();
  unsigned long long spent;
  do {
    __builtin_amdgcn_s_sleep(64);
    spent = wall_clock64() - t0;
  } while (scalar_load_coherent(y.flag) == y.epoch && spent < (unsigned long long)left);
  left = spent < (unsigned long long)left ? left - (uint32_t)spent : 0u;
}

constexpr uint32_t kPreSpinCap = 1u << 22;   // polls of `pre` before the last worker reports failure
constexpr uint32_t kProgressLost = 0xFFFFFFFFu;

// What the relay's fetch-and-add returned (in parts), once it has left it in `pre`.  The relay
// stores it right after that fetch-and-add, whose effect the caller has seen in the counter, so
// the wait is short and ends whatever the relay does next; the cap is a backstop that reports
// failure instead of hanging.
__device__ __forceinline__ uint32_t progress_at_request(const PtbCtl &c) {
  for (uint32_t spin = 0; spin < kPreSpinCap; ++spin) {
    const unsigned long long pre = __hip_atomic_load(c.pre, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)(pre >> 32) == c.epoch) return (uint32_t)pre;
    __builtin_amdgcn_s_sleep(2);
  }
  return kProgressLost;
}

// Logical blocks in parts.  A grid of fewer blocks than there are workers leaves most of them
// without work while the others take a whole block's time; where the workers are enough for it
// the counter therefore hands out PX * PY parts of each block (Sub's own, smaller blocks), and
// every worker takes at most one.  To the host nothing changes: progress is in whole blocks, and
// a request still lets every block that was begun be finished: the parts of the block in which
// the request fell that were not handed out before it are handed out after it, to workers that
// would otherwise leave (there are as many fetches as parts, so all of them are).
template <class SubBody, uint32_t PX, uint32_t PY>
struct PartsBody {
  using Sub = SubBody;
  using Args = typename Sub::Args;
  static constexpr int THREADS = Sub::THREADS;
  static constexpr int MIN_WAVES = Sub::MIN_WAVES;
  static constexpr unsigned DYN_LDS = Sub::DYN_LDS;
  static constexpr uint32_t PARTS_X = PX, PARTS = PX * PY;
  static_assert(kCoverPieces % PARTS == 0, "a part is a whole number of recorded pieces");
};
// The same for the last blocks of a grid that does not divide by the workers: each worker takes
// `whole` whole blocks (one fetch of PARTS parts each), then parts, so that the last round, in
// which most workers would find nothing, takes a part's time.  Nothing depends on the order in
// which the workers get there: a fetch of PARTS that comes after another worker's first part
// runs what it got part by part.
template <class WholeBody, class SubBody, uint32_t PX, uint32_t PY>
struct TailBody : PartsBody<SubBody, PX, PY> {
  using Whole = WholeBody;
  static constexpr int MIN_WAVES = Whole::MIN_WAVES;
  static constexpr unsigned DYN_LDS = Whole::DYN_LDS > SubBody::DYN_LDS ? Whole::DYN_LDS : SubBody::DYN_LDS;
};

// The team of this worker, and how many workers it has.
__device__ __forceinline__ uint32_t team_of(const PtbCtl &c) {
  const uint32_t t = blockIdx.x / kTeamSize;
  return t < c.team_count ? t : c.team_count - 1;
}
__device__ __forceinline__ uint32_t team_size(const PtbCtl &c, uint32_t team) {
  return team + 1 < c.team_count ? kTeamSize : c.workers - team * kTeamSize;
}
// Bodies whose workers may form teams: the others' kernels have none of this in them.
template <class Body, class = void>
struct HasTeams : std::false_type {};
template <class Body>
struct HasTeams<Body, std::enable_if_t<Body::TEAMS>> : std::true_type {};
// A worker's fetch of `add` task indices: what the counter held.
template <bool TEAMS>
__device__ __forceinline__ uint32_t fetch(const PtbCtl &c, uint32_t add) {
  if (!TEAMS || c.team_count == 0)
    return __hip_atomic_fetch_add(c.counter, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  unsigned long long *word = &c.teams[team_of(c)].word;
  for (;;) {
    const unsigned long long got = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t n = (uint32_t)got;
    if (n < kTeamBatch) return (uint32_t)(got >> 32) + n * add;
    if (n == kTeamBatch) {
      const uint32_t raw = __hip_atomic_fetch_add(c.counter, kTeamBatch * add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(word, (unsigned long long)raw << 32 | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return raw;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// One fetch of `add` parts: the parts [first, last) to run, none if last <= first.
__device__ __forceinline__ uint2 fetch_parts(const PtbCtl &c, uint32_t add, uint32_t P) {
  uint32_t idx = __hip_atomic_fetch_add(c.counter, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - c.counter_base;
  uint32_t end = c.limit;
  if (idx & kPreemptStep) {
    idx -= kPreemptStep;
    const uint32_t at = progress_at_request(c);
    end = at == kProgressLost ? 0u : (at + P - 1) / P * P;
  }
  return make_uint2(idx, idx + add < end ? idx + add : end);
}

// part `idx` of the grid (counted in parts)
template <class Body>
__device__ __forceinline__ void run_part(const typename Body::Args &args, const PtbCtl &c, const YieldCtl &y, uint32_t idx) {
  using Sub = typename Body::Sub;
  constexpr uint32_t P = Body::PARTS, PX = Body::PARTS_X, PY = P / PX;
  const uint32_t block = idx / P, part = idx % P;
  uint32_t bx, by, bz;
  delinearize(block, c.gx, c.gy, bx, by, bz);
  if constexpr (Sub::YIELDS) Sub::run_yielding(args, bx * PX + part % PX, by * PY + part / PX, bz, y);
  else Sub::run_be(args, bx * PX + part % PX, by * PY + part / PX, bz);
  record_part(c.cover, block, part, P, bx, by, bz, c.segment, blockIdx.x);
}
__device__ __forceinline__ YieldCtl yield_ctl(const PtbCtl &c, bool look_first) {
  return YieldCtl{c.flag_copies + (blockIdx.x % kFlagCopies) * kFlagCopyStride, c.epoch,
                  c.flag_copies != nullptr ? c.yield_ticks : 0u, c.yield_mask, look_first};
}

template <class Body>
__device__ __forceinline__ void ptb_parts(const typename Body::Args &args, const PtbCtl &c) {
  __shared__ uint2 s_got;
  if (threadIdx.x == 0) s_got = fetch_parts(c, 1, Body::PARTS);
  __syncthreads();
  const uint32_t idx = __builtin_amdgcn_readfirstlane(s_got.x), end = __builtin_amdgcn_readfirstlane(s_got.y);
  if (idx < end) run_part<Body>(args, c, yield_ctl(c, false), idx);
}

template <class Body>
__device__ __forceinline__ void ptb_tail(const typename Body::Args &args, const PtbCtl &c) {
  constexpr uint32_t P = Body::PARTS;
  __shared__ uint2 s_got[2];
  for (uint32_t it = 0;; ++it) {
    if (threadIdx.x == 0) s_got[it & 1] = fetch_parts(c, it < c.whole ? P : 1, P);
    __syncthreads();
    uint32_t idx = __builtin_amdgcn_readfirstlane(s_got[it & 1].x);
    const uint32_t end = __builtin_amdgcn_readfirstlane(s_got[it & 1].y);
    if (idx >= end) break;
    if (idx % P == 0 && end - idx == P) {
      uint32_t bx, by, bz;
      delinearize(idx / P, c.gx, c.gy, bx, by, bz);
      Body::Whole::run_yielding(args, bx, by, bz, yield_ctl(c, false));
      record(c.cover, idx / P, bx, by, bz, c.segment, blockIdx.x);
    } else {
      for (; idx < end; ++idx) run_part<Body>(args, c, yield_ctl(c, true), idx);
    }
  }
}

template <class Body>
__device__ __forceinline__ void ptb_blocks(const typename Body::Args &args, const PtbCtl &c) {
  __shared__ uint32_t s_idx[2];
  const uint32_t worker = blockIdx.x;
  // One lane fetches and broadcasts through LDS, so the exit decision is uniform over the
  // workgroup.  An index at or beyond `limit` means: grid exhausted, or a request folded
  // into the counter; either way the worker leaves, and what it fetched before is done.
  for (uint32_t it = 0;; ++it) {
    if (threadIdx.x == 0) s_idx[it & 1] = fetch<HasTeams<Body>::value>(c, c.chunk) - c.counter_base;
    __syncthreads();
    const uint32_t index = __builtin_amdgcn_readfirstlane(s_idx[it & 1]);
    if (index >= c.limit) break;  // uniform across the workgroup
    const uint32_t first = block_at(c, index), n = index < c.last_from ? c.chunk : c.last_chunk;
    const uint32_t last = c.end - first < n ? c.end : first + n;
    if constexpr (Body::RANGE) {
      // the blocks a fetch brought, handed to the body together (one-dimensional grids)
      if (last - first > 1) {
        Body::run_range(args, first, last);
        for (uint32_t idx = first; idx < last; ++idx) record(c.cover, idx, idx, 0, 0, c.segment, worker);
        if (c.single_pass) break;
        continue;
      }
    }
    for (uint32_t idx = first; idx < last; ++idx) {
      uint32_t bx, by, bz;
      delinearize(idx, c.gx, c.gy, bx, by, bz);
      if constexpr (Body::YIELDS)
        Body::run_yielding(args, bx, by, bz, yield_ctl(c, idx != first));
      else
        Body::run_be(args, bx, by, bz);
      record(c.cover, idx, bx, by, bz, c.segment, worker);
      // the paper ends every iteration with a barrier so that a worker handles one block
      // at a time; a body whose waves share no state across blocks does not need it
      if (Body::END_BARRIER) __syncthreads();
    }
    // the first fetches of all workers cover what is left: a second one could only fail
    if (c.single_pass) break;
  }
}

// A worker leaves: the last one of the segment publishes the progress to the host.
// All of this is relaxed on purpose: an agent- or system-scope release here would make
// every worker write back its whole L2 (tens of microseconds with a dirty output
// tile).  Ordering comes from data dependence instead: a worker adds to `exited` only
// after its last counter fetch has returned, so when the last worker sees the target
// every other fetch has been performed, and it reads the counter after that.  Kernel
// outputs become visible to the host at the end of the kernel as usual; the status
// word only says that the workers are gone.
template <bool TEAMS, bool PARTS>
__device__ __forceinline__ void ptb_leave(const PtbCtl &c) {
  if (threadIdx.x == 0) {
    if (TEAMS && c.team_count) {
      const uint32_t team = team_of(c);
      TeamLine &t = c.teams[team];
      if (__hip_atomic_fetch_add(&t.left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 != team_size(c, team)) return;
      __hip_atomic_store(&t.left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&t.word, kTeamIdle, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // (before the team counts as gone: whoever sees that may hand the line to another job)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    uint32_t old = __hip_atomic_fetch_add(c.exited, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1 == c.exit_target) {
      const uint32_t raw = __hip_atomic_load(c.counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t ctr = raw - c.counter_base;
      uint32_t progress = ctr < c.limit ? ctr : c.limit;
      // a request was folded in: the progress is what the relay's fetch-and-add returned
      if (ctr & kPreemptStep) progress = progress_at_request(c);
      if (progress != kProgressLost) progress = PARTS ? (progress + c.parts - 1) / c.parts : block_at(c, progress);   // every begun block is done
      // (both words carry the epoch and need no order, hence no round trip to the host between them)
      const unsigned long long tag = (unsigned long long)c.epoch << 32;
      __hip_atomic_store(c.host_status, tag | progress, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(c.host_raw, tag | raw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}
template <class Body, class = void>
struct HasParts : std::false_type {};
template <class Body>
struct HasParts<Body, std::void_t<typename Body::Sub>> : std::true_type {};
template <class Body, class = void>
struct HasWhole : std::false_type {};
template <class Body>
struct HasWhole<Body, std::void_t<typename Body::Whole>> : std::true_type {};
template <class Body>
__device__ __forceinline__ void ptb_body(const typename Body::Args &args, const PtbCtl &c) {
  if constexpr (HasWhole<Body>::value) ptb_tail<Body>(args, c);
  else if constexpr (HasParts<Body>::value) ptb_parts<Body>(args, c);
  else ptb_blocks<Body>(args, c);
  ptb_leave<HasTeams<Body>::value, HasParts<Body>::value>(c);
}
template <class Body>
__global__ __launch_bounds__(Body::THREADS, Body::MIN_WAVES) void ptb_kernel(typename Body::Args args, PtbCtl c) {
  ptb_body<Body>(args, c);
}

// Marker: stores a value into a pinned host word once earlier work on the stream is done.
__global__ void marker_kernel(uint32_t *word, uint32_t value) {
  if (threadIdx.x == 0)
    __hip_atomic_store(word, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One idle wave that stays on the GPU for `ticks` of the 100 MHz clock and then leaves
// (what a stream is kept busy with while its effect on another stream is measured).
__global__ void hold_kernel(uint32_t ticks) {
  const unsigned long long t0 = wall_clock64();
  while (wall_clock64() - t0 < (unsigned long long)ticks) __builtin_amdgcn_s_sleep(32);
}

// Every team's line as its last worker leaves it.
__global__ void team_init_kernel(TeamLine *t, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) { t[i].word = kTeamIdle; t[i].left = 0u; }
}

__global__ void set_word_kernel(uint32_t *word, uint32_t value) {
  if (threadIdx.x == 0)
    __hip_atomic_store(word, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A launch by the runtime's own call.  The <<<>>> form stores the configuration, fetches it again in the
// kernel's stub and then makes this call, and hipGetLastError is a third: 2.2 us against 2.0, of which a request
// of nine kernels has nine in a row.
template <class... P>
inline hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, hipStream_t s, P... p) {
  void *args[] = {&p...};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, args, lds, s);
  if (e != hipSuccess) (void)hipGetLastError();           // (reported here, not by whoever asks next)
  return e;
}

}  // namespace tally
