// sim_device.hpp -- gfx950 kernels of the scheduler simulator (device code).
//
// What every kernel shares (the parameters and limits of a launch), and the
// simulation of one instance by a workgroup of W waves (k_simulate_group, see
// group_exchange) for running sets beyond one wave's 1024 runs.  An instance that a
// single wave holds is simulated by the code of sim_wave.hpp, a batch of tiny ones by
// that of sim_tiny.hpp; prepare.hpp checks and ranks the requests beforehand.
//
// State of a workgroup's simulation:
//   running set R    -- ROWS x 64 register slots a wave, row r lane j holds one run:
//                       planned end Rend = p + est, x = s - p + t_r, completion
//                       C = p + o, key = est << 17 | rank, and h = f(Rend) +
//                       Rend - t_r, where f(c) is the planned memory at step c of
//                       all runs whose planned end is >= c (equation (2) summed
//                       over the planned set).  t_r is a base step that keeps the
//                       int32 values small (rebased every 2^16 steps).
//   fresh waiting F  -- two-level bitmap over key ranks in LDS; the smallest
//                       waiting key is the first set bit.  Its word is cached in
//                       scalar registers until it empties.
//   cancelled V      -- A_min: a register row U of recent cancellations in
//                       front of an unsorted (key, s | o << 16) array in LDS
//                       (or global memory), the smallest key found by a wave
//                       min-reduction; A_l: an append-only queue of promoted
//                       requests in global memory read through a register
//                       window.
// Per step: arrivals set bits of F; runs with C == t complete (A_l: runs still
// present at their planned end are promoted to the back of the queue); for
// A_min the projected memory P at t+1 is compared with M and runs are
// cancelled in ascending key while P > M; then candidates (smallest key of F,
// U and V; A_l: F first) are admitted while equation (2) holds.  The admission
// test needs only O(1) wave reductions because the planned set before the test
// is always feasible (every checkpoint after the candidate's planned end was
// verified when its runs were admitted), so it checks: step t (runs completing
// now hold s+o), step t+1 when a run is already past its planned end, every
// existing planned end <= the candidate's via max h, and the candidate's own
// planned end.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "schedsim.h"
#include "wave.hpp"

namespace sk {

// global-memory (address space 1) views of device arrays
typedef __attribute__((address_space(1))) int32_t g_i32;
typedef __attribute__((address_space(1))) uint64_t g_u64;

constexpr int kIdxBits = 17;
constexpr uint32_t kIdxMask = (1u << kIdxBits) - 1u;
constexpr int32_t kEstLimit = 1 << 15;
constexpr int32_t kPromptLimit = 1 << 16;
constexpr int32_t kRebase = 1 << 16;
constexpr int64_t kCapLimit = int64_t(1) << 30;

struct Params {
  int32_t K;
  int32_t max_requests;
  int64_t N;
  const int64_t* offsets;
  const int32_t* arrival;
  const int32_t* prompt;
  const int32_t* output;
  const int32_t* lower;
  const int32_t* upper;
  const int32_t* priority;
  const int32_t* tie_key;   // NULL: equal keys by index; else by (tie key, index)
  int32_t* completion;
  int32_t* evictions;
  int64_t* total_latency;
  int32_t* makespan;
  int64_t* request_steps;
  int64_t* total_evictions;
  int32_t* status;
  int32_t* algo_used;    // optional output: the policy each instance ran
  int32_t M;
  int64_t step_cap;      // > 0: user cap for every instance
  // workspace
  uint32_t* sort_a;
  uint32_t* sort_b;
  uint2* rec;
  int32_t* rank_of;
  int32_t* u_of_rank;    // A_l: u of the request at each rank (the workspace of the second sort buffer)
  int32_t* cap;
  int32_t* algo_of;      // adaptive runs: the policy each instance runs (else NULL)
  // with tie keys: each request's rank in tie order (its identity inside the
  // kernels, in place of the index), the inverse map, and staging arrays of
  // the per-request outputs indexed by that rank (copied out in index order
  // at the end)
  int32_t* tr_of;
  int32_t* idx_of;
  int32_t* comp_st;
  int32_t* ev_st;
  // cancelled set in global memory (the last retry pass): n entries per instance
  uint64_t* vglob;
  // LDS layout of k_simulate
  int32_t nw_max;        // 64-bit words of the level-0 bitmap
  int32_t nw1_max;       // 64-bit words of the level-1 bitmap
  int32_t cap_v;         // evicted-set capacity (LDS passes)
  int32_t retry_status;  // status for an outgrown running set: a later pass (kRetryRows) or SCHED_E_UNSUPPORTED
  int32_t retry_v_status;// status for an outgrown evicted set: a later pass (kRetryV) or SCHED_E_UNSUPPORTED
  int32_t run_mask;      // retry passes: bit 0 runs kRetryRows instances, bit 1 kRetryV ones
  int32_t run_cap;       // retry passes: most runs at once (a caller's forced capacity), else INT32_MAX
  // completion steps staged in LDS after the cancelled set (n_max slots) and
  // written out coalesced at the end of an instance
  int32_t stage_comp;
  // workgroup passes with global cancelled sets: n_max entries per wave of
  // each workgroup of the launch
  uint64_t* vgroup;
  // A_min with upper bounds (alone or in the adaptive policy): each instance's
  // issue-priority class (0-2 by the width of its intervals; 3: none), or -1
  // when all instances share a class
  int32_t* pclass;
  // A_min batches served in several rounds of waves: the order in which the
  // first launch takes the instances (longest expected first), built from a
  // key per instance and kOrderBuckets counters (then the buckets' cursors)
  int32_t* order;
  int32_t* okey;
  int32_t* obucket;
};

// Retry passes over a list (k_simulate_group_listed): the instances that the pass
// takes, their number, and a cursor over them.
struct RetryList {
  int32_t* list;
  int32_t* count;  // [0] the number, [1] the cursor
  int32_t room;    // entries that the list holds
};

// Whether some request of the instance of n > 0 requests from b on arrives after
// step 0 (arrivals do not decrease).  Where none does, every rank waits from the
// start, and k_prepare writes no rank_of.
__device__ __forceinline__ bool late_arrivals(const Params& P, const int64_t b, const int n) {
  return P.arrival && P.arrival[b + n - 1] > 0;
}

// words of the retry passes' counts: two a pass, eight passes a policy, two policies
constexpr int kRetryCounts = 32;

// buckets of the launch-order key
constexpr int kOrderBuckets = 64;

// Internal statuses of an instance handed to a later pass: its running set
// outgrew the register rows, or its cancelled set outgrew its slots.  The
// later pass simulates it again from step 0 with more room.
constexpr int kRetryRows = -100;
constexpr int kRetryV = -101;

// Whether a retry pass takes an instance of this status.
__device__ __forceinline__ bool retry_takes(const Params& P, const int status) {
  return (status == kRetryRows && (P.run_mask & 1)) || (status == kRetryV && (P.run_mask & 2));
}

// ---------------------------------------------------------------------------
// k_simulate
// ---------------------------------------------------------------------------
// r_end of an empty slot of the running set (below every planned end)
constexpr int32_t kEmpty = INT32_MIN;
// r_c of an empty slot (after every step)
constexpr int32_t kNever = 0x7FFFFFFF;

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int32_t>(v)));
}

// Status of a one-wave body that handed its state over (sim_wave.hpp) instead of ending.
constexpr int kResume = -102;

// The row ladders: the body above each rung (0: none).  The narrow ladder
// is 2, 3, 5, 8, 10; the wide one continues with 12 and 16.
__host__ __device__ constexpr int ladder_up(int rows, int top) {
  return rows >= top ? 0
         : rows == 2 ? 3 : rows == 3 ? 5 : rows == 5 ? 8 : rows == 8 ? 10 : rows == 10 ? 12 : rows == 12 ? 16 : 0;
}
// A body shrinks to the smallest rung that holds its runs with this many
// slots to spare (hysteresis: a shrink is never followed at once by a grow).
constexpr int kShrinkSpare = 16;
// A_min: at the start of a step, a register row of recent cancellations that
// holds more than this many entries goes to the LDS set
constexpr int kURowFlush = 48;

// ---------------------------------------------------------------------------
// A workgroup of W waves simulating one instance.  Every wave holds its
// own ROWS register rows of the running set (W x 64 x ROWS slots) and its own
// copy of the rest of the state (the bitmaps and the cancelled set in an LDS
// block of its own, the scalars, the register row of recent cancellations),
// which it updates exactly as the other waves do.  What depends on the whole
// running set is agreed at exchanges: each wave writes its partial results
// (a wave reduction over its rows), a barrier, and lane j < W of every wave
// reads wave j's partials, which one fold inside a 16-lane row combines.  A
// branch around an exchange depends only on state that every wave holds
// alike, so every wave reaches the same exchanges in the same order.  A new
// run goes to the wave that holds the fewest (counts kept alike in every
// wave: lane j holds wave j's).
// ---------------------------------------------------------------------------
// 64-bit LDS words before the waves' blocks: two alternating exchange buffers
// of W x 8 32-bit words, and for the policies whose runs may complete before
// their planned end (A_max, A_l) a list of each wave's completions at a step
// (W x 64 x ROWS entries).
__host__ __device__ constexpr int group_pre_words(int algo, int w, int rows) {
  return 8 * w + ((algo == SCHED_AMAX || algo == SCHED_AELL) ? w * 64 * rows : 0);
}

// A workgroup barrier that orders LDS accesses only (pending global stores
// are not waited for).
__device__ __forceinline__ void group_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One exchange of four 32-bit words per wave (two with `b`): lane j < W gets
// wave j's words; lanes >= W get their own wave's.  The two buffers alternate,
// so a wave can be at most one exchange ahead of another while it writes.
template <int W>
__device__ __forceinline__ uint4 group_exchange(uint4* red, int& par, int wv, int lane, uint4 a, uint4* b = nullptr) {
  uint4* buf = red + par * 2 * W;
  if (lane == 0) {
    buf[wv] = a;
    if (b) buf[W + wv] = *b;
  }
  group_barrier();
  par ^= 1;
  const int j = lane < W ? lane : wv;
  if (b) *b = buf[W + j];
  return buf[j];
}

// Folds over the lanes of the first 16-lane row (lanes >= W hold neutral values).
__device__ __forceinline__ uint32_t lanes_min_u32(uint32_t v) {
  return uniform_u32(wave::fold_in_row(v, wave::OpMinU32{}));
}
__device__ __forceinline__ int32_t lanes_max_i32(int32_t v) {
  return wave::uniform(static_cast<int32_t>(wave::fold_in_row(static_cast<uint32_t>(v), wave::OpMaxI32{})));
}
__device__ __forceinline__ int32_t lanes_sum_i32(int32_t v) {
  return wave::uniform(static_cast<int32_t>(wave::fold_in_row(static_cast<uint32_t>(v), wave::OpAddU32{})));
}

// Simulates instance k (whose validation status is st0) on a workgroup of W
// waves with ROWS register rows each (see group_exchange) and writes its outputs.  A
// running set that outgrows the rows ends the simulation with `retry_status` (the
// per-request outputs are then reset).  A cancelled set that outgrows its P.cap_v LDS
// slots ends it with P.retry_v_status; with VGLOBAL the set lives in global memory (n
// slots a wave, the most it can hold).
template <int ALGO, int ROWS, bool VGLOBAL, int W>
__device__ __forceinline__ void sim_instance(const Params& P, const int k, const int st0, const int retry_status) {
  static_assert(W > 1 && W <= 16, "one wave alone is wave_instance's");
  // only A_min and A_l have cancelled (or promoted) requests waiting: for the
  // other policies every head is fresh, and the code of the cancelled set is
  // left out of their kernels
  constexpr bool kHasV = ALGO == SCHED_AMIN || ALGO == SCHED_AELL;
  extern __shared__ uint64_t lds64[];
  const int lane = static_cast<int>(threadIdx.x & 63u);
  const int wv = wave::uniform(static_cast<int32_t>(threadIdx.x >> 6));
  const int64_t b = P.offsets[k];
  const int n = st0 == SCHED_OK ? static_cast<int>(P.offsets[k + 1] - b) : 0;
  const int32_t M = P.M;

  int status = st0;
  // counters live in vector registers (see wave::in_vgpr)
  int64_t rsteps = wave::in_vgpr<int64_t>(0);
  int64_t tot_ev = wave::in_vgpr<int64_t>(0);

  if (st0 == SCHED_OK && n > 0) {
    // each wave's block (bitmaps, cancelled set) follows the exchange
    // area, and the staged completion steps (one array for the workgroup)
    // follow the blocks; a global cancelled set has n entries per wave
    const int gstride = P.nw_max + P.nw1_max + (VGLOBAL ? 0 : P.cap_v);
    uint64_t* const lw = lds64 + group_pre_words(ALGO, W, ROWS) + wv * gstride;
    uint64_t* L0 = lw;
    uint64_t* L1 = lw + P.nw_max;
    // cancelled requests, one 64-bit entry each.  A_min: key | (s | o << 16) << 32,
    // slots [0, nVe) may start now, [nVe, nV) were cancelled at this step.
    // A_l: a FIFO ring of id | s << 17 | o << 33 | u << 48 from slot v_head.
    // (global: each wave of workgroup g has the n_max entries at
    // P.vgroup + (g W + wave) n_max; the workgroup simulates its instances
    // one after the other)
    uint64_t* vent = VGLOBAL ? P.vgroup + (static_cast<int64_t>(blockIdx.x) * W + wv) * P.max_requests
                             : L1 + P.nw1_max;
    // A_l: every request is promoted at most once, so its queue is an
    // append-only array of n entries in global memory (the instance's slice
    // of the workspace), read through a 64-entry register window
    constexpr bool kQueue = ALGO == SCHED_AELL;
    g_u64* qg = kQueue ? (g_u64*)(P.vglob + b) : nullptr;
    const int32_t cap_v = (VGLOBAL || kQueue) ? n : P.cap_v;
    int32_t* lcomp = reinterpret_cast<int32_t*>(lds64 + group_pre_words(ALGO, W, ROWS) + W * gstride);
    const bool stage_c = P.stage_comp != 0;
    const int nw = (n + 63) >> 6;
    const int nw1 = (nw + 63) >> 6;
    for (int w = lane; w < nw; w += 64) L0[w] = 0;
    for (int w = lane; w < nw1; w += 64) L1[w] = 0;
    if (stage_c)
      for (int i = static_cast<int>(threadIdx.x); i < n; i += 64 * W) lcomp[i] = -1;
    __syncthreads();
    // the exchange buffers, the completion lists, the run counts
    uint4* const gred = reinterpret_cast<uint4*>(lds64);
    uint64_t* const glist = lds64 + 8 * W + wv * 64 * ROWS;
    int gpar = 0;
    int32_t occ = 0;

    const int32_t cap = P.cap[k];
    // array bases in vector registers
    // array bases in vector registers, typed as global memory: plain pointers
    // would compile to flat accesses, and a flat store or atomic holds the
    // LDS wait counter until its global write completes, so every later LDS
    // wait of the wave would also wait for it
    auto base = [](auto* p) { return wave::in_vgpr(p); };
    const g_u64* rec = base((const g_u64*)(P.rec + b));  // (key, s | o << 16) as one 64-bit word
    const g_i32* arrival = P.arrival ? base((const g_i32*)(P.arrival + b)) : nullptr;
    const g_i32* rank_of = base((const g_i32*)(P.rank_of + b));
    const bool late = late_arrivals(P, b, n);
    const g_i32* upper_k = ALGO == SCHED_AELL ? (const g_i32*)(P.u_of_rank + b) : nullptr;  // by rank
    // per-request outputs by id (with tie keys: the staging arrays)
    // completion steps by id: staged in LDS after the cancelled set when the
    // launch has room for them (written out coalesced at the end of the
    // instance), else straight to the global outputs.  One generic pointer,
    // so the staged case costs no registers (its stores are flat stores to
    // LDS; the global case's are flat stores too, which measured the same)
    int32_t* cdst = base(P.stage_comp ? lcomp
                                      : (P.tie_key ? P.comp_st : P.completion) + b);
    g_i32* evictions = P.evictions ? base((g_i32*)((P.tie_key ? P.ev_st : P.evictions) + b)) : nullptr;

    // running set: register rows; an empty slot has r_end = kEmpty, r_c = kNever,
    // r_key = ~0, which every scan below treats as neutral, so scans cover all rows
    // (A_l also keeps each run's u, its planning length after a promotion)
    int32_t r_end[ROWS], r_x[ROWS], r_c[ROWS], r_h[ROWS], r_u[ROWS];
    uint32_t r_key[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      r_end[r] = kEmpty; r_x[r] = 0; r_c[r] = kNever; r_h[r] = 0; r_key[r] = 0xFFFFFFFFu; r_u[r] = 0;
    }
    int fr_row = 0;               // row that receives new runs ...
    uint64_t fr_mask = ~0ull;     // ... and its free lanes
    int32_t N = 0;                // number of runs
    int32_t X = 0;                // sum of x over runs
    int32_t t_r = 0;              // base step of x and h
    int32_t next_c = kNever;      // lower bound on the earliest completion step

    int32_t aw_base = -64, aw_a = 0x7FFFFFFF, aw_rank = 0, arr_ptr = 0;
    int32_t next_a = 0;           // arrival step of request arr_ptr (0: look at step 0)
    int32_t f_rank = -1, fw_base = -1;
    uint64_t f_word = 0ull;       // the bitmap word of f_rank (its LDS copy may still hold taken bits)
    uint32_t f_key = 0xFFFFFFFFu, f_so = 0, fw_key = 0xFFFFFFFFu, fw_so = 0;
    int32_t f_u = 0, fw_u = 0;
    int32_t nV = 0, nVe = 0, v_pos = -1, v_head = 0;
    uint32_t v_key = 0xFFFFFFFFu, v_so = 0;
    int32_t v_u = 0;
    // A_l: queue entries [vw_base, vw_base + 64) in lane order (entries
    // appended inside the window are written to it as well)
    uint32_t vw_lo = 0, vw_hi = 0;
    int32_t vw_base = -(1 << 30);
    // A_min: requests cancelled recently wait in a register row first (lane j
    // holds one: key and s | o << 16; u_gate is ~0 in the lanes filled at this
    // step, which may not start before the next one), with its smallest
    // startable entry cached in uh_*; a full row goes to the LDS set at the
    // start of a step.  Requests are usually started again within a step or
    // two of their cancellation, so most starts find their request here
    // without a scan of the LDS set.
    uint32_t u_key = 0xFFFFFFFFu, u_so = 0, u_gate = 0;
    uint64_t u_used = 0ull;
    uint32_t uh_key = 0xFFFFFFFFu, uh_so = 0;
    int32_t uh_lane = -1;
    int32_t n_done = 0;
    // the head cannot start before retry_at; valid until the next event
    int32_t retry_at = 0;
    int32_t t = 0;
    int32_t DT = 0;               // memory held at t by the runs completing at t

#define SK_LOAD_ARRIVALS()                                                           \
  do {                                                                               \
    aw_base = arr_ptr;                                                               \
    const int i_ = aw_base + lane;                                                   \
    aw_a = 0x7FFFFFFF;                                                               \
    aw_rank = 0;                                                                     \
    if (i_ < n) {                                                                    \
      aw_a = arrival ? arrival[i_] : 0;                                              \
      aw_rank = late ? rank_of[i_] : i_;                                             \
    }                                                                                \
  } while (0)
    // the record of fresh rank f_rank from the 64-record window (reloaded when
    // f_rank leaves it)
#define SK_F_RECORD()                                                                \
  do {                                                                               \
    if (fw_base < 0 || f_rank < fw_base || f_rank >= fw_base + 64) {                 \
      fw_base = f_rank;                                                              \
      const int rr_ = fw_base + lane;                                                \
      fw_key = 0xFFFFFFFFu;                                                          \
      fw_so = 0u;                                                                    \
      if (rr_ < n) {                                                                 \
        const uint64_t rv_ = rec[rr_];                                               \
        fw_key = static_cast<uint32_t>(rv_);                                         \
        fw_so = static_cast<uint32_t>(rv_ >> 32);                                    \
        if (ALGO == SCHED_AELL) fw_u = upper_k[rr_];                                 \
      }                                                                              \
    }                                                                                \
    f_key = wave::readlane_u(fw_key, f_rank - fw_base);                              \
    f_so = wave::readlane_u(fw_so, f_rank - fw_base);                                \
    if (ALGO == SCHED_AELL) f_u = wave::readlane(fw_u, f_rank - fw_base);            \
  } while (0)
    // smallest waiting fresh request: first set bit of the two-level bitmap in
    // LDS; its word stays in scalar registers (f_word) while it has bits left
#define SK_F_FIND()                                                                  \
  do {                                                                               \
    const uint64_t w1_ = lane < nw1 ? L1[lane] : 0ull;                               \
    const uint64_t nz_ = wave::ballot(w1_ != 0ull);                                  \
    if (nz_ == 0ull) {                                                               \
      f_rank = -1;                                                                   \
      f_key = 0xFFFFFFFFu;                                                           \
    } else {                                                                         \
      const int j1_ = __builtin_ctzll(nz_);                                          \
      const uint64_t w1v_ = wave::readlane_u64(w1_, j1_);                            \
      const int j0_ = j1_ * 64 + __builtin_ctzll(w1v_);                              \
      f_word = uniform_u64(L0[j0_]);                                                 \
      f_rank = j0_ * 64 + __builtin_ctzll(f_word);                                   \
      SK_F_RECORD();                                                                 \
    }                                                                                \
  } while (0)
    // f_rank starts: it is the lowest bit of f_word.  The next one is the next
    // bit of the same word (no LDS access); an emptied word is written back
    // and leaves the summary level, and the search goes to the next word.
#define SK_F_TAKE()                                                                  \
  do {                                                                               \
    f_word &= f_word - 1ull;                                                         \
    if (f_word != 0ull) {                                                            \
      f_rank = (f_rank & ~63) + __builtin_ctzll(f_word);                             \
      SK_F_RECORD();                                                                 \
    } else {                                                                         \
      const int j0_ = f_rank >> 6;                                                   \
      if (lane == 0) {                                                               \
        L0[j0_] = 0ull;                                                              \
        atomicAnd(reinterpret_cast<unsigned long long*>(&L1[j0_ >> 6]), ~(1ull << (j0_ & 63))); \
      }                                                                              \
      SK_F_FIND();                                                                   \
    }                                                                                \
  } while (0)
    // per-lane smallest cancelled entry over slots [FROM_, TO_): vb_k, vb_p, vb_s.
    // The loop runs over blocks of 128 slots with a uniform trip count (no
    // per-lane exit), both loads of a block in flight at once; a slot past
    // TO_ reads the last slot instead and counts as empty.
#define SK_V_SCAN(FROM_, TO_)                                                        \
  uint32_t vb_k = 0xFFFFFFFFu, vb_s = 0u;                                            \
  int32_t vb_p = -1;                                                                 \
  for (int b_ = (FROM_); b_ < (TO_); b_ += 128) {                                    \
    const int to_ = (TO_), last_ = to_ - 1;                                          \
    const int j0_ = b_ + lane, j1_ = b_ + 64 + lane;                                 \
    const uint64_t e0_ = vent[j0_ < last_ ? j0_ : last_];                            \
    const uint64_t e1_ = vent[j1_ < last_ ? j1_ : last_];                            \
    const uint32_t k0_ = j0_ < to_ ? static_cast<uint32_t>(e0_) : 0xFFFFFFFFu;       \
    const uint32_t k1_ = j1_ < to_ ? static_cast<uint32_t>(e1_) : 0xFFFFFFFFu;       \
    const bool l0_ = k0_ < vb_k;                                                     \
    vb_k = l0_ ? k0_ : vb_k;                                                         \
    vb_p = l0_ ? j0_ : vb_p;                                                         \
    vb_s = l0_ ? static_cast<uint32_t>(e0_ >> 32) : vb_s;                            \
    const bool l1_ = k1_ < vb_k;                                                     \
    vb_k = l1_ ? k1_ : vb_k;                                                         \
    vb_p = l1_ ? j1_ : vb_p;                                                         \
    vb_s = l1_ ? static_cast<uint32_t>(e1_ >> 32) : vb_s;                            \
  }
    // smallest cancelled request that may start now (slots [0, nVe))
#define SK_V_FIND()                                                                  \
  do {                                                                               \
    SK_V_SCAN(0, nVe)                                                                \
    const uint32_t kv_ = wave::min_u32_all(vb_k);                                    \
    const uint64_t at_ = wave::ballot(vb_k == kv_);                                  \
    const uint32_t km_ = wave::uniform_u(kv_);                                       \
    v_key = km_;                                                                     \
    v_pos = -1;                                                                      \
    if (km_ != 0xFFFFFFFFu) {                                                        \
      const int ln_ = __builtin_ctzll(at_);                                          \
      v_pos = wave::readlane(vb_p, ln_);                                             \
      v_so = wave::readlane_u(vb_s, ln_);                                            \
    }                                                                                \
  } while (0)
    // the requests cancelled at the previous step may start now: merge them
    // into the cached head instead of rescanning every slot
#define SK_V_MERGE()                                                                 \
  do {                                                                               \
    SK_V_SCAN(nVe, nV)                                                               \
    const uint32_t kv_ = wave::min_u32_all(vb_k);                                    \
    const uint64_t at_ = wave::ballot(vb_k == kv_);                                  \
    const uint32_t km_ = wave::uniform_u(kv_);                                       \
    if (km_ < v_key) {                                                               \
      const int ln_ = __builtin_ctzll(at_);                                          \
      v_key = km_;                                                                   \
      v_pos = wave::readlane(vb_p, ln_);                                             \
      v_so = wave::readlane_u(vb_s, ln_);                                            \
    }                                                                                \
    nVe = nV;                                                                        \
  } while (0)
    // A_l: the oldest promoted request (head of the queue), planned with u.
    // The window moves to the head when the head leaves it; the fence makes
    // the lane-0 appends visible to the other lanes' loads.
#define SK_V_HEAD()                                                                  \
  do {                                                                               \
    v_pos = -1;                                                                      \
    v_key = 0xFFFFFFFFu;                                                             \
    if (nV > 0) {                                                                    \
      if (v_head - vw_base >= 64 || v_head < vw_base) {                              \
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");                       \
        vw_base = v_head;                                                            \
        const int j_ = v_head + lane;                                                \
        const uint64_t w_ = j_ < n ? static_cast<uint64_t>(qg[j_]) : 0ull;           \
        vw_lo = static_cast<uint32_t>(w_);                                           \
        vw_hi = static_cast<uint32_t>(w_ >> 32);                                     \
      }                                                                              \
      const int d_ = v_head - vw_base;                                               \
      const uint64_t e_ = (static_cast<uint64_t>(wave::readlane_u(vw_hi, d_)) << 32) | \
                          wave::readlane_u(vw_lo, d_);                               \
      const uint32_t ix_ = static_cast<uint32_t>(e_) & kIdxMask;                     \
      const uint32_t s_ = static_cast<uint32_t>(e_ >> 17) & 0xFFFFu;                 \
      const uint32_t o_ = static_cast<uint32_t>(e_ >> 33) & 0x7FFFu;                 \
      v_u = static_cast<int32_t>((e_ >> 48) & 0x7FFFu);                              \
      v_pos = v_head;                                                                \
      v_key = (static_cast<uint32_t>(v_u) << kIdxBits) | ix_;                        \
      v_so = s_ | (o_ << 16);                                                        \
    }                                                                                \
  } while (0)
    // A_min: the smallest startable entry of the register row
#define SK_U_FIND()                                                                  \
  do {                                                                               \
    const uint32_t uk_ = u_key | u_gate;                                             \
    const uint32_t um_ = wave::min_u32_all(uk_);                                     \
    const uint64_t ua_ = wave::ballot(uk_ == um_);                                   \
    uh_key = wave::uniform_u(um_);                                                   \
    uh_lane = -1;                                                                    \
    if (uh_key != 0xFFFFFFFFu) {                                                     \
      uh_lane = __builtin_ctzll(ua_);                                                \
      uh_so = wave::readlane_u(u_so, uh_lane);                                       \
    }                                                                                \
  } while (0)
    // the head of the waiting set: smaller key of the fresh and cancelled heads
    // (A_l: every fresh request comes before the promoted ones); derived where
    // it is used rather than carried through the loop
#define SK_PICK()                                                                    \
  const bool c_fromU = ALGO == SCHED_AMIN && uh_key < v_key;                         \
  const uint32_t vh_key = c_fromU ? uh_key : v_key;                                  \
  const uint32_t vh_so = c_fromU ? uh_so : v_so;                                     \
  const bool c_any = f_rank >= 0 || (kHasV && (v_pos >= 0 || c_fromU));              \
  const bool c_fromF = !kHasV || (f_rank >= 0 && (ALGO == SCHED_AELL || f_key < vh_key)); \
  const uint32_t c_key = c_fromF ? f_key : vh_key;                                   \
  const uint32_t c_so = c_fromF ? f_so : vh_so;                                      \
  const int32_t c_s = static_cast<int32_t>(c_so & 0xFFFFu);                          \
  const int32_t c_o = static_cast<int32_t>(c_so >> 16);                              \
  const int32_t c_est = ALGO == SCHED_ARANDOM ? c_o : static_cast<int32_t>(c_key >> kIdxBits); \
  const int32_t c_u = c_fromF ? f_u : v_u;
    // BODY with the compile-time row index r equal to the uniform row RR_
#define SK_AT_ROW(RR_, BODY)                                                         \
  _Pragma("unroll") for (int r = 0; r < ROWS; ++r) {                                 \
    if (r == (RR_)) {                                                                \
      BODY                                                                           \
    }                                                                                \
  }
    // A run with raw planned end ek and x = xk leaves: every run with
    // t+1 < Rend <= ek loses its share of f at its own planned end.
#define SK_DROP_SHARE(T_, XK_, EK_)                                                  \
  do {                                                                               \
    const int32_t tt_ = (T_), ek_ = (EK_);                                           \
    if (ek_ > tt_ + 1) {                                                             \
      const uint32_t lo_ = static_cast<uint32_t>(tt_) + 2u;                          \
      const uint32_t span_ = static_cast<uint32_t>(ek_) - lo_;                       \
      const uint32_t dx_ = static_cast<uint32_t>(XK_) - static_cast<uint32_t>(t_r);  \
      _Pragma("unroll") for (int r_ = 0; r_ < ROWS; ++r_) {                          \
        const uint32_t e_ = static_cast<uint32_t>(r_end[r_]);                        \
        const bool in_ = e_ - lo_ <= span_;                                          \
        r_h[r_] = static_cast<int32_t>(static_cast<uint32_t>(r_h[r_]) - (in_ ? dx_ + e_ : 0u)); \
      }                                                                              \
    }                                                                                \
  } while (0)

    // Issue priority among the waves of a SIMD: the more requests an instance
    // still has to complete, the higher (four levels by the unfinished
    // fraction), so the instances that bound the launch are not slowed by
    // their SIMD-mates; where a batch mixes interval widths (A_min with upper
    // bounds), the static class of the instance and whether half of it is
    // done instead.  Outputs do not depend on it.
    int prio = -1;
    const int pcls = (ALGO == SCHED_AMIN && P.pclass) ? P.pclass[k] : -1;
#define SK_SET_PRIORITY()                                                            \
  do {                                                                               \
    const int lv_ = pcls >= 0 ? pcls + (2 * (n - n_done) > n ? 1 : 0) : (4 * (n - n_done) - 1) / n; \
    if (lv_ != prio) {                                                               \
      prio = lv_;                                                                    \
      if (lv_ >= 3) __builtin_amdgcn_s_setprio(3);                                   \
      else if (lv_ == 2) __builtin_amdgcn_s_setprio(2);                              \
      else if (lv_ == 1) __builtin_amdgcn_s_setprio(1);                              \
      else __builtin_amdgcn_s_setprio(0);                                            \
    }                                                                                \
  } while (0)
    SK_SET_PRIORITY();
    for (;;) {
      if (t > cap) {
        status = SCHED_E_STEP_CAP;
        break;
      }
      if (t - t_r >= kRebase) {
        const uint32_t d = static_cast<uint32_t>(t - t_r);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          r_x[r] = static_cast<int32_t>(static_cast<uint32_t>(r_x[r]) + d);
          r_h[r] = static_cast<int32_t>(static_cast<uint32_t>(r_h[r]) - d);
        }
        X += N * static_cast<int32_t>(d);
        t_r = t;
      }
      bool heads_changed = false;
      bool event = false;
      // ---- 1. arrivals; requests cancelled at the previous step become eligible
      if (t >= next_a) {
        // the cached word goes back to LDS before arrivals set bits in it
        if (f_rank >= 0 && lane == 0) L0[f_rank >> 6] = f_word;
        while (arr_ptr < n) {
          if (arr_ptr >= aw_base + 64) SK_LOAD_ARRIVALS();
          const bool take = (aw_base + lane >= arr_ptr) && aw_a <= t;
          const uint64_t m = wave::ballot(take);
          if (m == 0ull) break;
          if (take) {
            atomicOr(reinterpret_cast<unsigned long long*>(&L0[aw_rank >> 6]), 1ull << (aw_rank & 63));
            atomicOr(reinterpret_cast<unsigned long long*>(&L1[aw_rank >> 12]), 1ull << ((aw_rank >> 6) & 63));
          }
          arr_ptr += __builtin_popcountll(m);
          if (arr_ptr < aw_base + 64) break;
        }
        if (arr_ptr < n) {
          if (arr_ptr >= aw_base + 64) SK_LOAD_ARRIVALS();
          next_a = wave::readlane(aw_a, arr_ptr - aw_base);
        } else {
          next_a = 0x7FFFFFFF;
        }
        SK_F_FIND();
        heads_changed = true;
      }
      if (ALGO == SCHED_AMIN && nVe != nV) {
        SK_V_MERGE();
        heads_changed = true;
      }
      if (ALGO == SCHED_AMIN && u_used != 0ull) {
        const int cnt = __builtin_popcountll(u_used);
        const bool fresh_u = wave::ballot(u_gate != 0u) != 0ull;  // cancelled at the last step
        if (cnt > kURowFlush) {
          // the row goes to the LDS set (every entry of it may start now)
          if (nV + cnt > cap_v) {
            status = P.retry_v_status;
            break;
          }
          const bool mine = (u_used >> lane) & 1ull;
          const int slot = nV + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                   static_cast<uint32_t>(u_used >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(u_used), 0u)));
          if (mine) vent[slot] = (static_cast<uint64_t>(u_so) << 32) | u_key;
          const uint32_t k_ = u_key;
          u_key = 0xFFFFFFFFu;
          u_gate = 0u;
          u_used = 0ull;
          // its smallest entry competes with the LDS set's head
          const uint32_t um_ = wave::min_u32_all(mine ? k_ : 0xFFFFFFFFu);
          const uint64_t ua_ = wave::ballot(mine && k_ == um_);
          const uint32_t mk_ = wave::uniform_u(um_);
          if (mk_ < v_key) {
            const int ln_ = __builtin_ctzll(ua_);
            v_key = mk_;
            v_so = wave::readlane_u(u_so, ln_);
            v_pos = wave::readlane(slot, ln_);
          }
          nV += cnt;
          nVe = nV;
          uh_key = 0xFFFFFFFFu;
          uh_lane = -1;
          heads_changed = true;
        } else if (fresh_u) {
          u_gate = 0u;
          SK_U_FIND();
          heads_changed = true;
        }
      }
      if (heads_changed) event = true;

      // ---- 2. completions at t; DT = memory they still hold at t (s + o each)
      DT = 0;
      if (t >= next_c) {
        int32_t sx = 0;
        int ndone = 0;
        int lc = 0;                    // this wave's completions listed
        uint32_t gcmin = 0xFFFFFFFFu;  // the next event, agreed
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          const bool hit = r_c[r] == t;
          const uint64_t m = wave::ballot(hit);
          if (m) {
            ndone += __builtin_popcountll(m);
            if constexpr (ALGO == SCHED_AMAX || ALGO == SCHED_AELL) {
              // every wave drops the shares of every wave's completions: list them
              if (hit) {
                const int pos = lc + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                         static_cast<uint32_t>(m >> 32),
                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
                glist[pos] = static_cast<uint64_t>(static_cast<uint32_t>(r_x[r])) |
                             (static_cast<uint64_t>(static_cast<uint32_t>(r_end[r])) << 32);
              }
              lc += __builtin_popcountll(m);
            } else if (ALGO == SCHED_AMAX || ALGO == SCHED_AELL) {
              // planned with u >= o: the run may end before its planned end
              uint64_t mm = m;
              while (mm) {
                const int ln = __builtin_ctzll(mm);
                mm &= mm - 1;
                SK_DROP_SHARE(t, wave::readlane(r_x[r], ln), wave::readlane(r_end[r], ln));
              }
            }
            if (hit) cdst[r_key[r] & kIdxMask] = t;
            sx += hit ? r_x[r] : 0;
            r_end[r] = hit ? kEmpty : r_end[r];
            r_c[r] = hit ? kNever : r_c[r];
            r_key[r] = hit ? 0xFFFFFFFFu : r_key[r];
            if (r == fr_row) fr_mask |= m;
          }
        }
        {
          // agree on the completions (and, but for A_l, the next one)
          uint32_t cl = 0xFFFFFFFFu;
          if constexpr (ALGO != SCHED_AELL) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              const uint32_t ev = static_cast<uint32_t>(r_c[r]);
              cl = ev < cl ? ev : cl;
            }
            cl = wave::min_u32(cl);
          }
          const uint4 g = group_exchange<W>(gred, gpar, wv, lane,
                                            make_uint4(static_cast<uint32_t>(ndone), static_cast<uint32_t>(wave::sum_i32(sx)),
                                                       cl, static_cast<uint32_t>(lc)));
          const int32_t nd_j = lane < W ? static_cast<int32_t>(g.x) : 0;
          occ -= nd_j;
          const int32_t nd = lanes_sum_i32(nd_j);
          const int32_t sxw = lanes_sum_i32(lane < W ? static_cast<int32_t>(g.y) : 0);
          gcmin = lanes_min_u32(lane < W ? g.z : 0xFFFFFFFFu);
          if constexpr (ALGO == SCHED_AMAX || ALGO == SCHED_AELL) {
            if (lanes_sum_i32(lane < W ? static_cast<int32_t>(g.w) : 0) > 0) {
              for (int j = 0; j < W; ++j) {
                const int cj = wave::readlane(static_cast<int32_t>(g.w), j);
                const uint64_t* lj = lds64 + 8 * W + j * 64 * ROWS;
                for (int e0 = 0; e0 < cj; e0 += 64) {
                  const uint64_t ev = e0 + lane < cj ? lj[e0 + lane] : 0ull;
                  const int ne = cj - e0 < 64 ? cj - e0 : 64;
                  for (int q = 0; q < ne; ++q) {
                    const int32_t xq = wave::readlane(static_cast<int32_t>(static_cast<uint32_t>(ev)), q);
                    const int32_t eq = wave::readlane(static_cast<int32_t>(ev >> 32), q);
                    SK_DROP_SHARE(t, xq, eq);
                  }
                }
              }
              group_barrier();  // every wave has read the lists: they may be written again
            }
          }
          if (nd) {
            event = true;
            X -= sxw;
            N -= nd;
            DT = sxw + nd * (t - t_r);
            n_done += nd;
            SK_SET_PRIORITY();
          }
        }
        // ---- 3. done?
        if (n_done == n) break;
        // ---- 3'. A_l: a run still present at its planned end t (planned with
        // l, so o > l) is promoted: it leaves, plans with u and joins the back of
        // the queue, lowest index first among this step's promotions
        if (ALGO == SCHED_AELL) {
          bool promoted = false;
          {
          for (;;) {
            uint32_t best = 0xFFFFFFFFu;
            int32_t brow = 0;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              const uint32_t kk = r_end[r] == t ? (r_key[r] & kIdxMask) : 0xFFFFFFFFu;
              const bool lt = kk < best;
              best = lt ? kk : best;
              brow = lt ? r : brow;
            }
            const uint32_t iv = wave::min_u32_all(best);
            const uint64_t at = wave::ballot(best == iv);
            // the smallest index over the waves; its wave removes the run (the
            // exchange that finds nothing left to promote also agrees on the
            // next event)
            const uint32_t il = wave::uniform_u(iv);
            int ln = 0, rr = 0;
            int32_t xk = 0, ck = 0, uk = 0;
            uint32_t kk = 0;
            if (il != 0xFFFFFFFFu) {
              ln = __builtin_ctzll(at);
              rr = wave::readlane(brow, ln);
              SK_AT_ROW(rr, xk = wave::readlane(r_x[r], ln); ck = wave::readlane(r_c[r], ln);
                        uk = wave::readlane(r_u[r], ln); kk = wave::readlane_u(r_key[r], ln);)
            }
            uint32_t cl = 0xFFFFFFFFu;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              const uint32_t ev = static_cast<uint32_t>(r_c[r]), pe = static_cast<uint32_t>(r_end[r]);
              cl = ev < cl ? ev : cl;
              cl = pe < cl ? pe : cl;
            }
            uint4 g2 = make_uint4(kk, wave::min_u32(cl), 0u, 0u);
            const uint4 g = group_exchange<W>(gred, gpar, wv, lane,
                                              make_uint4(il, static_cast<uint32_t>(xk), static_cast<uint32_t>(ck),
                                                         static_cast<uint32_t>(uk)), &g2);
            const uint32_t gi = lane < W ? g.x : 0xFFFFFFFFu;
            const uint32_t imin = lanes_min_u32(gi);
            if (imin == 0xFFFFFFFFu) {
              gcmin = lanes_min_u32(lane < W ? g2.y : 0xFFFFFFFFu);
              break;
            }
            if (nV >= cap_v) {
              status = P.retry_v_status;
              break;
            }
            const int win = __builtin_ctzll(wave::ballot(gi == imin));
            xk = wave::readlane(static_cast<int32_t>(g.y), win);
            ck = wave::readlane(static_cast<int32_t>(g.z), win);
            uk = wave::readlane(static_cast<int32_t>(g.w), win);
            kk = wave::readlane_u(g2.x, win);
            if (wv == win) {
              SK_AT_ROW(rr, r_end[r] = wave::writelane(r_end[r], kEmpty, ln);
                        r_c[r] = wave::writelane(r_c[r], kNever, ln);
                        r_key[r] = wave::writelane_u(r_key[r], 0xFFFFFFFFu, ln);)
              if (rr == fr_row) fr_mask |= 1ull << ln;
            }
            occ -= lane == win ? 1 : 0;
            X -= xk;
            N -= 1;
            const int32_t pk = t - static_cast<int32_t>(kk >> kIdxBits);
            const uint64_t sk = static_cast<uint32_t>(xk - t_r + pk);
            const uint64_t okk = static_cast<uint32_t>(ck - pk);
            {
              // every wave appends the same entry; one counts the promotion
              const int slot = v_head + nV;
              const uint64_t qe = imin | (sk << 17) | (okk << 33) | (static_cast<uint64_t>(uk) << 48);
              if (lane == 0) {
                qg[slot] = qe;
                if (evictions && wv == 0)
                  __hip_atomic_fetch_add(&evictions[imin], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
              if (slot >= vw_base && slot - vw_base < 64) {
                vw_lo = wave::writelane_u(vw_lo, static_cast<uint32_t>(qe), slot - vw_base);
                vw_hi = wave::writelane_u(vw_hi, static_cast<uint32_t>(qe >> 32), slot - vw_base);
              }
            }
            ++nV;
            ++tot_ev;
            promoted = true;
          }
          }
          if (status != SCHED_OK) break;
          if (promoted) {
            event = true;
            if (v_pos < 0) SK_V_HEAD();
          }
        }
        // next event: a completion (A_l: or a planned end, where a run is promoted);
        // empty slots read as unsigned are above every step
        next_c = static_cast<int32_t>(gcmin);
      }

      // ---- 4. A_min: cancel in ascending (o~, index) while memory at t+1 > M
      if (ALGO == SCHED_AMIN) {
        int32_t Pm = X + N * (t + 1 - t_r);
        if (Pm > M) {
          while (Pm > M) {
            uint32_t best = r_key[0];
            int32_t brow = 0;
#pragma unroll
            for (int r = 1; r < ROWS; ++r) {
              const bool lt = r_key[r] < best;
              best = lt ? r_key[r] : best;
              brow = lt ? r : brow;
            }
            const uint32_t kv = wave::min_u32_all(best);
            const uint64_t at = wave::ballot(best == kv);
            uint32_t kmin = 0xFFFFFFFFu;
            int32_t ek = 0, xk = 0, ck = 0;
            {
              // the smallest key over the waves; its wave removes the run
              const uint32_t kl = wave::uniform_u(kv);
              int ln = 0, rr = 0;
              if (kl != 0xFFFFFFFFu) {
                ln = __builtin_ctzll(at);
                rr = wave::readlane(brow, ln);
                SK_AT_ROW(rr, ek = wave::readlane(r_end[r], ln); xk = wave::readlane(r_x[r], ln);
                          ck = wave::readlane(r_c[r], ln);)
              }
              const uint4 g = group_exchange<W>(gred, gpar, wv, lane,
                                                make_uint4(kl, static_cast<uint32_t>(ek), static_cast<uint32_t>(xk),
                                                           static_cast<uint32_t>(ck)));
              const uint32_t gk = lane < W ? g.x : 0xFFFFFFFFu;
              kmin = lanes_min_u32(gk);
              if (kmin == 0xFFFFFFFFu) {  // no run: impossible while P > M > 0
                status = SCHED_E_UNSUPPORTED;
                break;
              }
              if (u_used == ~0ull && nV >= cap_v) {
                status = P.retry_v_status;
                break;
              }
              const int win = __builtin_ctzll(wave::ballot(gk == kmin));
              ek = wave::readlane(static_cast<int32_t>(g.y), win);
              xk = wave::readlane(static_cast<int32_t>(g.z), win);
              ck = wave::readlane(static_cast<int32_t>(g.w), win);
              if (wv == win) {
                SK_AT_ROW(rr, r_end[r] = wave::writelane(r_end[r], kEmpty, ln);
                          r_c[r] = wave::writelane(r_c[r], kNever, ln);
                          r_key[r] = wave::writelane_u(r_key[r], 0xFFFFFFFFu, ln);)
                if (rr == fr_row) fr_mask |= 1ull << ln;
              }
              occ -= lane == win ? 1 : 0;
            }
            SK_DROP_SHARE(t, xk, ek);
            X -= xk;
            N -= 1;
            Pm -= xk + t + 1 - t_r;
            const int32_t oh = static_cast<int32_t>(kmin >> kIdxBits);
            const uint32_t idx = kmin & kIdxMask;
            const int32_t pk = ek - oh;
            const int32_t gen = t - pk;
            const int32_t nh = gen > oh ? gen : oh;
            const int32_t sk = xk - t_r + pk;
            const int32_t okk = ck - pk;
            const uint32_t so = static_cast<uint32_t>(sk) | (static_cast<uint32_t>(okk) << 16);
            const uint32_t nkey = (static_cast<uint32_t>(nh) << kIdxBits) | idx;
            if (u_used != ~0ull) {
              // into a free lane of the register row, startable from the next step
              const int ul = __builtin_ctzll(~u_used);
              u_key = wave::writelane_u(u_key, nkey, ul);
              u_so = wave::writelane_u(u_so, so, ul);
              u_gate = wave::writelane_u(u_gate, 0xFFFFFFFFu, ul);
              u_used |= 1ull << ul;
              if (lane == 0 && wv == 0 && evictions)
                __hip_atomic_fetch_add(&evictions[idx], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
              if (lane == 0) {
                vent[nV] = (static_cast<uint64_t>(so) << 32) | nkey;
                if (evictions && wv == 0)
                  __hip_atomic_fetch_add(&evictions[idx], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
              ++nV;
            }
            ++tot_ev;
          }
          if (status != SCHED_OK) break;
          event = true;
        }
      }
      if (event) retry_at = 0;

      // ---- 5. admission of the longest feasible prefix in key order
      bool stuck = true;          // the head cannot start before the next event
      int32_t wait_until = t + 1; // otherwise: not before this step
      for (;;) {
        SK_PICK();
        if (!c_any) break;
        const int32_t s = c_s, est = c_est;
        const int32_t E = t + est;
        const int32_t tp1 = t + 1;
        // step t+1: every running request is present; exact when a planned end
        // falls there and implied by the first planned end after it otherwise
        const int32_t Pm = X + N * (tp1 - t_r);
        if (Pm + s + 1 > M) break;
        stuck = false;
        if (t < retry_at) {
          wait_until = retry_at;
          break;
        }
        // step t (runs completing at t hold s+o); implied by step t+1 when DT = 0
        if (DT > 0 && DT + X + N * (t - t_r) + s > M) break;
        // planned ends c in (t+1, E] need h + t_r - t + s <= M (h + t_r = f(c) + c);
        // the candidate's own end E needs f(E) + s + est <= M, f(E) = sum of x + E - t_r
        const uint32_t lo2 = static_cast<uint32_t>(t) + 2u;
        const bool win = E > tp1;
        const uint32_t span = win ? static_cast<uint32_t>(E) - lo2 : 0u;
        const int32_t cE = E - t_r;
        const int32_t lim = win ? M + t - t_r - s : 0x7FFFFFFF;  // h above this violates
        int32_t fl = 0, hmx = INT32_MIN;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          const int32_t e = r_end[r];
          const bool in = static_cast<uint32_t>(e) - lo2 <= span;
          const int32_t hv = in ? r_h[r] : INT32_MIN;
          hmx = hv > hmx ? hv : hmx;
          fl += e >= E ? r_x[r] + cE : 0;
        }
        {
          // one exchange agrees on both conditions and on the step to retry at
          // (both ways of failing are prepared, see below)
          int32_t fix = 0, emin = kNever;
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            const int32_t a = r_h[r] - lim, bb = r_end[r] - 1 - t;
            const int32_t m = a < bb ? a : bb;
            const bool in = static_cast<uint32_t>(r_end[r]) - lo2 <= span;
            fix = (in && r_h[r] > lim && m > fix) ? m : fix;
            const int32_t e = r_end[r];
            emin = (e >= E && e < emin) ? e : emin;
          }
          const uint4 g = group_exchange<W>(
              gred, gpar, wv, lane,
              make_uint4(static_cast<uint32_t>(wave::max_i32(hmx)), static_cast<uint32_t>(wave::sum_i32(fl)),
                         static_cast<uint32_t>(wave::max_i32(fix)), wave::min_u32(static_cast<uint32_t>(emin))));
          const int32_t hg = lanes_max_i32(lane < W ? static_cast<int32_t>(g.x) : INT32_MIN);
          const int32_t fg = lanes_sum_i32(lane < W ? static_cast<int32_t>(g.y) : 0);
          if (hg > lim || (win && fg + s + est > M)) {
            if (hg > lim)
              retry_at = t + lanes_max_i32(lane < W ? static_cast<int32_t>(g.z) : 0);
            else
              retry_at = static_cast<int32_t>(lanes_min_u32(lane < W ? g.w : 0xFFFFFFFFu)) - est + 1;
            wait_until = retry_at;
            break;
          }
          // passed: the test below (one wave's) then passes with f = fg
          fl = lane == 0 ? fg : 0;
          hmx = INT32_MIN;
        }
        // both conditions in one ballot: the sum is left in every lane, so the
        // passing case costs a single vector-to-scalar hand-off
        const int32_t fv = wave::sum_i32_all(fl);
        const bool end_bad = win && fv + s + est > M;
        if (wave::ballot(hmx > lim || end_bad)) {
          if (wave::ballot(hmx > lim)) {
            // each violating end improves by one per step, or leaves the window
            int32_t fix = 0;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              const int32_t a = r_h[r] - lim, bb = r_end[r] - 1 - t;
              const int32_t m = a < bb ? a : bb;
              const bool in = static_cast<uint32_t>(r_end[r]) - lo2 <= span;
              fix = (in && r_h[r] > lim && m > fix) ? m : fix;
            }
            retry_at = t + wave::max_i32(fix);
          } else {
            // f at the sliding end only grows until it passes the next planned end
            int32_t emin = kNever;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              const int32_t e = r_end[r];
              emin = (e >= E && e < emin) ? e : emin;
            }
            retry_at = static_cast<int32_t>(wave::min_u32(static_cast<uint32_t>(emin))) - est + 1;
          }
          wait_until = retry_at;
          break;
        }
        const int32_t f = wave::uniform(fv);
        // admit: start at p = t; runs whose planned end is in (t+1, E] gain its share
        // a free slot first: without one nothing has changed for this candidate
        int owner = 0;  // the wave that takes the run
        {
          // the wave with the fewest runs (the lowest such); all full: outgrown
          const uint32_t oc = lane < W ? (static_cast<uint32_t>(occ) << 4) | static_cast<uint32_t>(lane) : 0xFFFFFFFFu;
          const uint32_t om = lanes_min_u32(oc);
          if (static_cast<int>(om >> 4) >= 64 * ROWS) {
            status = retry_status;
            break;
          }
          owner = static_cast<int>(om & 15u);
          occ += lane == owner ? 1 : 0;
          if (wv == owner && fr_mask == 0ull) {
            // it has a free slot (its count is below its rows' slots)
            int rr = 0;
            uint64_t mm = 0ull;
#pragma unroll
            for (int r = ROWS - 1; r >= 0; --r) {
              const uint64_t m = wave::ballot(r_end[r] == kEmpty);
              rr = m ? r : rr;
              mm = m ? m : mm;
            }
            fr_row = rr;
            fr_mask = mm;
          }
        }
        const int32_t xw = s - t + t_r;
        const int32_t hw = f + (xw + cE) + cE;
        if (win) {
          const uint32_t dh = static_cast<uint32_t>(xw) - static_cast<uint32_t>(t_r);
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            const uint32_t e = static_cast<uint32_t>(r_end[r]);
            r_h[r] = static_cast<int32_t>(static_cast<uint32_t>(r_h[r]) + (e - lo2 <= span ? e + dh : 0u));
          }
        }
        {
          const int32_t cw = t + c_o;
          if (wv == owner) {
          const int ln = __builtin_ctzll(fr_mask);
          fr_mask &= fr_mask - 1;
          const uint32_t kw = c_key;
          const int32_t uw = c_u;
          SK_AT_ROW(fr_row, r_end[r] = wave::writelane(r_end[r], E, ln); r_x[r] = wave::writelane(r_x[r], xw, ln);
                    r_c[r] = wave::writelane(r_c[r], cw, ln); r_key[r] = wave::writelane_u(r_key[r], kw, ln);
                    r_h[r] = wave::writelane(r_h[r], hw, ln);
                    if (ALGO == SCHED_AELL) r_u[r] = wave::writelane(r_u[r], uw, ln);)
          }
          const int32_t ew = ALGO == SCHED_AELL && E < cw ? E : cw;  // A_l: promotion at E
          next_c = ew < next_c ? ew : next_c;
        }
        X += xw;
        N += 1;
        if (c_fromF) {
          SK_F_TAKE();
        } else if (ALGO == SCHED_AELL) {
          ++v_head;
          --nV;
          SK_V_HEAD();
        } else if (ALGO == SCHED_AMIN && c_fromU) {
          // from the register row
          u_key = wave::writelane_u(u_key, 0xFFFFFFFFu, uh_lane);
          u_used &= ~(1ull << uh_lane);
          SK_U_FIND();
        } else {
          // the last eligible entry moves into the hole; the last pending one fills
          // its place.  Lane 0 and lane 1 do the two moves with one read and one
          // write (when the hole is the last eligible slot, only the second move
          // is left, as in doing them one after the other)
          if (lane < 2) {
            const int le = nVe - 1;
            const int src = lane == 0 ? le : nV - 1;
            const uint64_t mv = vent[src];
            const bool act = lane == 0 ? v_pos != le : nV > nVe;
            if (act) vent[lane == 0 ? v_pos : le] = mv;
          }
          --nVe;
          --nV;
          SK_V_FIND();
        }
        stuck = true;
        wait_until = t + 1;
        retry_at = 0;
      }
      if (status != SCHED_OK) break;

      // ---- 6. this step processes every running request once
      rsteps += N;
      int32_t tn = t + 1;
      if (ALGO != SCHED_AMIN || (nV == nVe && !wave::ballot(u_gate != 0u))) {
        // Nothing changes before the next completion, arrival or (A_min)
        // overflow; until then the head cannot start before wait_until (or at
        // all when stuck: the memory at t+1 only grows).
        int32_t jump = stuck ? 0x7FFFFFFF : wait_until;
        jump = next_c < jump ? next_c : jump;
        jump = next_a < jump ? next_a : jump;
        if (ALGO == SCHED_AMIN && N > 0) {
          const int32_t Pm = X + N * (t + 1 - t_r);  // <= M here
          // first step whose projection exceeds M, if it comes before the jump
          if (static_cast<int64_t>(Pm) + static_cast<int64_t>(N) * (jump - 1 - t) > M) {
            const int32_t tev = t + (M - Pm) / N + 1;
            jump = tev < jump ? tev : jump;
          }
        }
        const int32_t lim = t_r + kRebase;
        jump = lim < jump ? lim : jump;
        jump = cap + 1 < jump ? cap + 1 : jump;
        if (jump > tn) {
          rsteps += static_cast<int64_t>(N) * (jump - tn);
          tn = jump;
        }
      }
      t = tn;
    }
  }

  // ---- epilogue: totals from the per-request outputs (with tie keys, first
  // copied from the staging arrays, by id, to the outputs, by index)
  __syncthreads();
  const bool keep = (status == SCHED_OK || status == SCHED_E_STEP_CAP) && n > 0;
  const bool tie = P.tie_key != nullptr;
  const bool st_c = P.stage_comp != 0;
  int64_t tel = 0, mk = 0;
  if (keep) {
    const int32_t* lc =
        reinterpret_cast<const int32_t*>(lds64 + group_pre_words(ALGO, W, ROWS) +
                                         W * (P.nw_max + P.nw1_max + (VGLOBAL ? 0 : P.cap_v)));
    for (int c = 0; c < n; c += 64 * W) {
      const int i = c + static_cast<int>(threadIdx.x);
      if (i < n) {
        const int32_t id = tie ? P.tr_of[b + i] : i;
        int32_t ci;
        if (st_c || tie) {
          ci = st_c ? lc[id] : P.comp_st[b + id];
          P.completion[b + i] = ci;
        } else {
          ci = P.completion[b + i];
        }
        if (P.evictions && tie) P.evictions[b + i] = P.ev_st[b + id];
        if (ci >= 0) {
          tel += ci - (P.arrival ? P.arrival[b + i] : 0);
          mk = ci > mk ? ci : mk;
        }
      }
    }
  } else if (status != st0 && n > 0) {
    // capacity outgrown at run time: report like an invalid instance (or hand
    // it to a retry pass, which starts from these values)
    int32_t* comp = tie ? P.comp_st : P.completion;
    int32_t* evs = tie ? P.ev_st : P.evictions;
    for (int c = 0; c < n; c += 64 * W) {
      const int i = c + static_cast<int>(threadIdx.x);
      if (i < n) {
        comp[b + i] = -1;
        if (P.evictions) evs[b + i] = 0;
      }
    }
  }
  tel = wave::sum_i64(tel);
  mk = wave::max_i64(mk);
  {
    // over the waves (the exchange area is free: every wave is past the
    // barrier above, so past its last exchange)
    int64_t* gt = reinterpret_cast<int64_t*>(lds64);
    if (lane == 0) {
      gt[2 * wv] = tel;
      gt[2 * wv + 1] = mk;
    }
    __syncthreads();
    tel = 0;
    mk = 0;
    for (int j = 0; j < W; ++j) {
      tel += gt[2 * j];
      mk = gt[2 * j + 1] > mk ? gt[2 * j + 1] : mk;
    }
  }
  if (!keep) {
    rsteps = 0;
    tot_ev = 0;
  }
  if (threadIdx.x == 0) {
    P.total_latency[k] = tel;
    if (P.makespan) P.makespan[k] = static_cast<int32_t>(mk);
    if (P.request_steps) P.request_steps[k] = rsteps;
    if (P.total_evictions) P.total_evictions[k] = tot_ev;
    P.status[k] = status;
  }
}

// A workgroup of W waves per instance, ROWS register rows each (W x 64 x ROWS
// runs): for few large instances, and for the instances whose running set
// outgrows one wave's rows (a retry pass).  With P.run_mask set, only the
// instances an earlier pass handed over run.
// Workgroup g simulates instances g, g + grid, ... (a launch with global
// cancelled sets has fewer workgroups than instances: each workgroup's sets
// are its own).
template <int ALGO, int W, int ROWS, bool VGLOBAL>
__global__ __launch_bounds__(64 * W) void k_simulate_group(Params P) {
  for (int k = blockIdx.x; k < P.K; k += gridDim.x) {
    if (P.algo_of && P.algo_of[k] != ALGO) continue;
    int st0 = P.status[k];
    if (P.run_mask) {
      if (!retry_takes(P, st0)) continue;
      st0 = SCHED_OK;
    }
    sim_instance<ALGO, ROWS, VGLOBAL, W>(P, k, st0, P.retry_status);
    __syncthreads();  // the next instance reuses the LDS
  }
}

// A retry pass of a large batch: a workgroup takes the next instance of R.list until none
// is left, since which instances of a batch need the pass may follow any pattern (a sweep
// has its parameters in blocks), and each takes milliseconds.  A list too short for them
// (only where offsets that decrease give the same requests to many instances) is not used.
// A kernel of its own: with the list in the other's loop, that took up to 6% longer (one
// A_min instance of 100000 on 4 waves 419 ms, not 394).
template <int ALGO, int W, bool VGLOBAL>
__global__ __launch_bounds__(64 * W) void k_simulate_group_listed(Params P, RetryList R) {
  extern __shared__ uint64_t lds64[];
  const bool listed = R.count[0] <= R.room;
  for (int g = blockIdx.x; listed || g < P.K; g += gridDim.x) {
    int k = g;
    if (listed) {
      if (threadIdx.x == 0) lds64[0] = static_cast<uint64_t>(atomicAdd(&R.count[1], 1));
      __syncthreads();
      k = wave::uniform(static_cast<int32_t>(lds64[0]));
      __syncthreads();  // the instance uses the LDS
      if (k >= R.count[0]) return;
      k = R.list[k];
    } else if ((P.algo_of && P.algo_of[k] != ALGO) || !retry_takes(P, P.status[k])) {
      continue;
    }
    sim_instance<ALGO, 16, VGLOBAL, W>(P, k, SCHED_OK, P.retry_status);
    __syncthreads();  // the next instance reuses the LDS
  }
}

// The workgroup kernels of a policy: EACH(...) instantiates them, with `extern` before
// it they are declared to the host code that launches them.  2 x 8 and 4 x 4 waves and rows
// (1024 runs) as a first launch, 4 x 16 and 8 x 16 (4096 and 8192 runs) as retry passes.
#define SK_GROUP_FIRST(EACH, ALGO, VGLOBAL)                                                \
  EACH template __global__ void k_simulate_group<ALGO, 2, 8, VGLOBAL>(Params);             \
  EACH template __global__ void k_simulate_group<ALGO, 4, 4, VGLOBAL>(Params);
#define SK_GROUP_RETRY(EACH, ALGO, W, VGLOBAL)                                             \
  EACH template __global__ void k_simulate_group<ALGO, W, 16, VGLOBAL>(Params);            \
  EACH template __global__ void k_simulate_group_listed<ALGO, W, VGLOBAL>(Params, RetryList);
#define SK_GROUP_KERNELS(EACH)                                                             \
  SK_GROUP_FIRST(EACH, SCHED_AMAX, false)                                                  \
  SK_GROUP_RETRY(EACH, SCHED_AMAX, 4, false)                                               \
  SK_GROUP_RETRY(EACH, SCHED_AMAX, 8, false)                                               \
  SK_GROUP_FIRST(EACH, SCHED_HSF, false)                                                   \
  SK_GROUP_RETRY(EACH, SCHED_HSF, 4, false)                                                \
  SK_GROUP_RETRY(EACH, SCHED_HSF, 8, false)                                                \
  SK_GROUP_RETRY(EACH, SCHED_ARANDOM, 4, false)                                            \
  SK_GROUP_RETRY(EACH, SCHED_ARANDOM, 8, false)                                            \
  SK_GROUP_RETRY(EACH, SCHED_AELL, 4, false)                                               \
  SK_GROUP_RETRY(EACH, SCHED_AELL, 8, false)
#define SK_GROUP_KERNELS_AMIN(EACH)                                                        \
  SK_GROUP_FIRST(EACH, SCHED_AMIN, false)                                                  \
  SK_GROUP_FIRST(EACH, SCHED_AMIN, true)                                                   \
  SK_GROUP_RETRY(EACH, SCHED_AMIN, 4, false)                                               \
  SK_GROUP_RETRY(EACH, SCHED_AMIN, 4, true)                                                \
  SK_GROUP_RETRY(EACH, SCHED_AMIN, 8, true)
#undef SK_SET_PRIORITY
#undef SK_LOAD_ARRIVALS
#undef SK_PICK
#undef SK_F_FIND
#undef SK_F_RECORD
#undef SK_F_TAKE
#undef SK_V_FIND
#undef SK_V_SCAN
#undef SK_V_MERGE
#undef SK_V_HEAD
#undef SK_U_FIND
#undef SK_AT_ROW
#undef SK_DROP_SHARE

}  // namespace sk

