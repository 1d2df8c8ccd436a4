// sim_wave.hpp -- one wave64 simulating one instance (device code of the
// one-wave kernels: k_simulate, k_simulate_ladder, k_simulate_ladder_roomy,
// k_simulate_ladder_wide).
//
// What bounds it: an instance is a serial chain of scheduling events
// (admissions, cancellations, promotions, completions), each a short chain of
// dependent instructions on one wave, and a lone wave issues one instruction
// per ~4 (independent) to ~8 (dependent) cycles, with ~30 where a vector result
// steers a branch.  So what counts is instructions and vector-to-scalar
// hand-offs per event, and the state is laid out for few of both:
//   running set R    -- ROWS x 64 register slots, row r lane j holds one run:
//                       planned end r_end = p + est, x = s - p + t_r (t_r: a
//                       base step, moved every 2^16 steps, that keeps x small),
//                       completion C = p + o, key = est << 17 | rank, and
//                       f = f(r_end), where f(c) is the planned memory at step c
//                       of all runs whose planned end is >= c (equation (2)
//                       summed over the planned set).  f is at most M in every
//                       slot, an empty one included, so a test of new values
//                       needs no mask.
//   fresh waiting F  -- two-level bitmap over key ranks in LDS; the first word
//                       with bits left is held in scalar registers, with the
//                       records of its 64 ranks in vector registers.
//   cancelled V      -- A_min: the 64 smallest (key, s | o << 16) entries, or
//                       fewer, sorted in a register row (lanes v_lo to v_hi),
//                       the rest sorted in LDS (or global memory) as a stack
//                       whose top is the smallest.  A request cancelled at step
//                       t waits in a pending row until t + 1.  Nine in ten
//                       cancelled requests belong among the first 16 entries
//                       (they are the next ones to start again), so an insertion
//                       is one compare, one lane shift and two lane writes, and
//                       the head costs nothing to find.
//                       A_l: an append-only queue of promoted requests in global
//                       memory, 64 entries of it in a register row.
// Both waiting sets thus offer their next candidates in lane order, and the
// admissions of a step take them from there four at a time: one pass over the
// rows and one transposed wave reduction give f at the planned ends of all four
// (wave::sum4).  When all four fit, one more pass gives the rows' new values of f
// and one ballot admits them; else each admission is one pass over the rows with
// new values of f, one ballot, and the write of the run into its slot.
// The benchmark's A_min batch (4096 x 1000) took 10.9 ms and H-SF's sweep (65536 x
// 2000) 33.7 ms when every admission did a reduction, the head's search and the
// test's second pass over the rows of its own; now 8.3 and 19.3 ms.
#pragma once

#include "sim_device.hpp"

namespace sk {

// A branch that the step loop rarely takes: the code behind it is placed out of
// the way, since a lone wave waits about 30 cycles for its instructions after
// every jump taken.
#define SK_RARE(COND) __builtin_expect(!!(COND), 0)
#define SK_USUAL(COND) __builtin_expect(!!(COND), 1)

// The loop-carried state of one instance, handed from one body to another with
// a different number of register rows (the row ladder: 2, 3, 5, 8, 10, then 12
// and 16 rows).  A body grows at an admission that finds no free slot (the next
// body's extra rows start empty) and shrinks, at the start of a step's
// admissions, once the running set fits a smaller body with room to spare (it
// first moves the runs of its upper rows into free slots of the lower ones).
// The LDS sets stay where they are.  `resume`: continue with the admissions of
// step t (false: start step t from its arrivals).
template <int SR>
struct WaveStateT {
  static constexpr int kRows = SR;
  int32_t r_end[SR], r_x[SR], r_c[SR], r_f[SR], r_u[SR];
  uint32_t r_key[SR];
  int fr_row;
  uint64_t fr_mask;
  int32_t N, X, t_r, next_c, aw_base, aw_a, aw_rank, arr_ptr, next_a;
  int32_t f_base, fw_u;
  uint32_t fw_key, fw_so;
  uint64_t f_word;
  uint32_t vw_key, vw_so, pn_key, pn_so;
  int32_t v_lo, v_hi, v_sp, n_pend, n_ovf;
  int32_t q_head, q_n, q_base;
  int32_t e_max, f_max;
  int32_t n_done, retry_at, t, DT;
  int64_t rsteps, tot_ev;
  int32_t next_rows;
  bool resume;
};
// the narrow ladder (up to 10 rows, four waves a SIMD) and the wide one (up
// to 16 rows, for few large instances and for instances that outgrow the
// narrow one)
using WaveState = WaveStateT<10>;
using WaveStateWide = WaveStateT<16>;

// The fresh set's bitmaps at the start: empty, or where every request arrives at
// step 0, full.  Returns the requests that need not arrive any more.
__device__ __forceinline__ int start_waiting(const Params& P, const int64_t b, const int n, uint64_t* L0, uint64_t* L1) {
  const int nw = (n + 63) >> 6, nw1 = (nw + 63) >> 6;
  const uint64_t all = n > 0 && !late_arrivals(P, b, n) ? ~0ull : 0ull;
  for (int w = threadIdx.x; w < nw; w += 64) L0[w] = w == nw - 1 ? all >> (63 - ((n - 1) & 63)) : all;
  for (int w = threadIdx.x; w < nw1; w += 64) L1[w] = w == nw1 - 1 ? all >> (63 - ((nw - 1) & 63)) : all;
  return all != 0ull ? n : 0;
}

// The state of an instance at step 0 (what a body starting fresh holds).
template <typename ST>
__device__ __forceinline__ void fresh_state(ST& st, const int arr_ptr) {
#pragma unroll
  for (int r = 0; r < ST::kRows; ++r) {
    st.r_end[r] = kEmpty; st.r_x[r] = 0; st.r_c[r] = kNever; st.r_f[r] = 0; st.r_key[r] = 0xFFFFFFFFu; st.r_u[r] = 0;
  }
  st.fr_row = 0; st.fr_mask = ~0ull; st.N = 0; st.X = 0; st.t_r = 0; st.next_c = kNever;
  st.aw_base = -64; st.aw_a = kNever; st.aw_rank = 0; st.arr_ptr = arr_ptr; st.next_a = 0;
  st.f_base = -1; st.fw_u = 0; st.fw_key = 0xFFFFFFFFu; st.fw_so = 0; st.f_word = 0ull;
  st.vw_key = threadIdx.x < 32 ? 0u : 0xFFFFFFFFu; st.vw_so = 0; st.pn_key = 0xFFFFFFFFu; st.pn_so = 0;
  st.v_lo = 32; st.v_hi = 32; st.v_sp = 0; st.n_pend = 0; st.n_ovf = 0;
  st.q_head = 0; st.q_n = 0; st.q_base = -(1 << 30); st.e_max = 0; st.f_max = 0;
  st.n_done = 0; st.retry_at = 0; st.t = 0; st.DT = 0; st.rsteps = 0; st.tot_ev = 0;
  st.next_rows = 2; st.resume = false;
}

// lanes [lo, hi) as a mask (0 <= lo <= hi <= 64)
__device__ __forceinline__ uint64_t lane_span(int lo, int hi) {
  return hi > lo ? (~0ull >> (64 - (hi - lo))) << lo : 0ull;
}

// Simulates instance k (whose validation status is st0) with ROWS register
// rows; the status it returns and the counters in *st go to finish_instance.
// A running set that outgrows the rows ends the simulation with
// `retry_status`, or, with TO_STATE, the state goes to *st and it returns
// kResume.  With FROM_STATE the body continues from *st instead of starting at step 0.  A
// cancelled set that outgrows its registers and P.cap_v LDS slots ends it with
// P.retry_v_status; with VGLOBAL the stack lives in global memory (n slots, the
// most it can hold).  CAPPED holds the running set to P.run_cap runs.
template <int ALGO, int ROWS, bool FROM_STATE = false, bool TO_STATE = false, bool VGLOBAL = false,
          bool CAPPED = false, typename ST = WaveState, bool CLS = true, bool PRIO = true>
__device__ __forceinline__ int wave_instance(const Params& P, const int k, const int st0, const int retry_status,
                                            ST* st) {
  constexpr int kStateRows = ST::kRows;
  static_assert(!(FROM_STATE || TO_STATE) || ROWS <= kStateRows, "state holds at most kStateRows rows");
  constexpr bool kAmin = ALGO == SCHED_AMIN;
  constexpr bool kQueue = ALGO == SCHED_AELL;
  // a run of these policies may complete before its planned end
  constexpr bool kEarly = ALGO == SCHED_AMAX || ALGO == SCHED_AELL;
  // every run completes at its planned end
  constexpr bool kOnPlan = ALGO == SCHED_HSF || ALGO == SCHED_ARANDOM;
  // Requests start in ascending planned length (but for arrivals), so a new run's
  // planned end is usually the latest.  f at such an end is known without a pass
  // over the rows and a wave reduction: with e_max and f_max kept, H-SF's sweep
  // (65536 x 2000) went from 27.9 to 22.4 ms and one A_max instance of 100000 from
  // 161 to 150 ms.
  constexpr bool kSorted = ALGO == SCHED_HSF || ALGO == SCHED_AMAX;
  // Four admissions in one test.  Not where each is cheap by itself and one in a few
  // steps is the rule: H-SF's sweep took 44 ms with attempts that mostly failed.
  constexpr bool kGroup = !kSorted;
  // nothing happens to the runs but their completions once nothing waits
  constexpr bool kDrains = kOnPlan || ALGO == SCHED_AMAX;
  extern __shared__ uint64_t lds64[];
  const int lane = static_cast<int>(threadIdx.x);
  const int64_t b = P.offsets[k];
  // a body that hands its state over only ever runs valid, non-empty instances
  const int n = (TO_STATE || st0 == SCHED_OK) ? static_cast<int>(P.offsets[k + 1] - b) : 0;
  const int32_t M = P.M;

  int status = st0;
  int handoff = 0;  // TO_STATE: rows of the body that continues (status kResume)
  // counters live in vector registers (see wave::in_vgpr)
  int64_t rsteps = wave::in_vgpr<int64_t>(FROM_STATE ? st->rsteps : 0);
  int64_t tot_ev = wave::in_vgpr<int64_t>(FROM_STATE ? st->tot_ev : 0);

  if (TO_STATE || (st0 == SCHED_OK && n > 0)) {
    uint64_t* L0 = lds64;
    uint64_t* L1 = lds64 + P.nw_max;
    // A_min: the stack of cancelled requests below the register row, one 64-bit
    // entry key | (s | o << 16) << 32 each, slots [0, v_sp) with the smallest on
    // top; pending entries beyond the pending row come down from the last slot
    uint64_t* vent = VGLOBAL ? P.vglob + b : L1 + P.nw1_max;
    const int32_t cap_v = VGLOBAL ? n : P.cap_v;
    // A_l: every request is promoted at most once, so its queue is an
    // append-only array of n entries id | s << 17 | o << 33 | u << 48 in global
    // memory (the instance's slice of the workspace)
    g_u64* qg = kQueue ? (g_u64*)(P.vglob + b) : nullptr;
    int32_t* lcomp = reinterpret_cast<int32_t*>(L1 + P.nw1_max + (VGLOBAL ? 0 : P.cap_v));
    const bool stage_c = P.stage_comp != 0;
    const int nw = (n + 63) >> 6;
    const int nw1 = (nw + 63) >> 6;
    int arr_ptr = 0;  // the next request to arrive
    if (!FROM_STATE) {
      arr_ptr = start_waiting(P, b, n, L0, L1);
      if (stage_c)
        for (int i = lane; i < n; i += 64) lcomp[i] = -1;
      __syncthreads();
    }
    const int32_t cap = P.cap[k];
    // array bases in vector registers, typed as global memory: plain pointers
    // would compile to flat accesses, and a flat store or atomic holds the
    // LDS wait counter until its global write completes, so every later LDS
    // wait of the wave would also wait for it
    auto base = [](auto* p) { return wave::in_vgpr(p); };
    const g_u64* rec = base((const g_u64*)(P.rec + b));  // (key, s | o << 16) as one 64-bit word
    const g_i32* arrival = P.arrival ? base((const g_i32*)(P.arrival + b)) : nullptr;
    const g_i32* rank_of = base((const g_i32*)(P.rank_of + b));
    const g_i32* upper_k = kQueue ? (const g_i32*)(P.u_of_rank + b) : nullptr;  // by rank
    // completion steps by id (with tie keys: the tie rank), staged in LDS after
    // the cancelled set when the launch has room for them (written out coalesced
    // at the end of the instance), else straight to the global outputs (with
    // tie keys: the staging arrays)
    const int32_t* cdst = base((P.tie_key ? P.comp_st : P.completion) + b);
    const int32_t* ev_at = base((P.tie_key ? P.ev_st : P.evictions) + b);
    // LDS offsets of the bitmap levels, the stack and the staged steps
    const uint32_t l0_at = wave::lds_offset(L0), l1_at = wave::lds_offset(L1);
    const uint32_t vs_at = l1_at + 8u * static_cast<uint32_t>(P.nw1_max), lc_at = wave::lds_offset(lcomp);
    auto v_store = [&](uint64_t mask, int at, uint64_t e) {
      if (VGLOBAL) wave::global_store64(mask, vent + at, e);
      else wave::lds_store64(mask, vs_at + 8u * static_cast<uint32_t>(at), e);
    };
    auto v_load = [&](int at) {
      if (VGLOBAL) wave::wait_stores();
      return vent[at];
    };

    // running set: an empty slot has r_end = kEmpty, r_c = kNever, r_key = ~0,
    // which every scan below treats as neutral, so scans cover all rows
    // (A_l also keeps each run's u, its planning length after a promotion)
    int32_t r_end[ROWS], r_x[ROWS], r_c[ROWS], r_f[ROWS], r_u[ROWS];
    uint32_t r_key[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      r_end[r] = kEmpty; r_x[r] = 0; r_c[r] = kNever; r_f[r] = 0; r_key[r] = 0xFFFFFFFFu; r_u[r] = 0;
      if (FROM_STATE) {
        r_end[r] = st->r_end[r]; r_x[r] = st->r_x[r]; r_c[r] = st->r_c[r];
        r_f[r] = st->r_f[r]; r_key[r] = st->r_key[r]; r_u[r] = st->r_u[r];
      }
    }
    int fr_row = 0;               // row that receives new runs ...
    uint64_t fr_mask = ~0ull;     // ... and its free lanes
    int32_t N = 0;                // number of runs
    int32_t X = 0;                // sum of x over runs
    int32_t t_r = 0;              // base step of x
    int32_t next_c = kNever;      // lower bound on the next completion (A_l: or promotion)
    int32_t aw_base = -64, aw_a = kNever, aw_rank = 0;
    int32_t next_a = 0;           // arrival step of request arr_ptr (0: look at step 0)
    // F: the waiting ranks of [f_base, f_base + 64) (none: no fresh request
    // waits) and their records; the LDS copy of the word may hold taken bits
    int32_t f_base = -1;
    uint64_t f_word = 0ull;
    uint32_t fw_key = 0xFFFFFFFFu, fw_so = 0;
    int32_t fw_u = 0;
    // A_min: the sorted register row (key 0 in the lanes below v_lo, ~0 in those
    // from v_hi on, so that one compare finds a key's place), the stack pointer, the pending row's count and the pending entries in LDS.
    // A_l: entries [q_base, q_base + 64) of the queue in lane order
    uint32_t vw_key = lane < 32 ? 0u : 0xFFFFFFFFu, vw_so = 0, pn_key = 0xFFFFFFFFu, pn_so = 0;
    int32_t v_lo = 32, v_hi = 32, v_sp = 0, n_pend = 0, n_ovf = 0;
    int32_t q_head = 0, q_n = 0, q_base = -(1 << 30);
    // kSorted: no run's planned end is above e_max, and f_max = f(e_max)
    int32_t e_max = 0, f_max = 0;
    int32_t n_done = 0;
    int32_t retry_at = 0;         // the head cannot start before it; valid until the next event
    int32_t t = 0;
    int32_t DT = 0;               // memory held at t by the runs completing at t
    if (FROM_STATE) {
      fr_row = st->fr_row; fr_mask = st->fr_mask; N = st->N; X = st->X; t_r = st->t_r; next_c = st->next_c;
      aw_base = st->aw_base; aw_a = st->aw_a; aw_rank = st->aw_rank; arr_ptr = st->arr_ptr; next_a = st->next_a;
      f_base = st->f_base; fw_key = st->fw_key; fw_so = st->fw_so; f_word = st->f_word;
      n_done = st->n_done; retry_at = st->retry_at; t = st->t; DT = st->DT;
      if constexpr (kAmin || kQueue) {
        vw_key = st->vw_key; vw_so = st->vw_so;
      }
      if constexpr (kAmin) {
        pn_key = st->pn_key; pn_so = st->pn_so; v_lo = st->v_lo; v_hi = st->v_hi; v_sp = st->v_sp;
        n_pend = st->n_pend; n_ovf = st->n_ovf;
      }
      if constexpr (kSorted) {
        e_max = st->e_max; f_max = st->f_max;
      }
      if constexpr (kQueue) {
        fw_u = st->fw_u; q_head = st->q_head; q_n = st->q_n; q_base = st->q_base;
      }
    }

#define SK_LOAD_ARRIVALS()                                                           \
  do {                                                                               \
    aw_base = arr_ptr;                                                               \
    const int i_ = aw_base + lane;                                                   \
    const int ic_ = i_ < n ? i_ : n - 1;                                             \
    aw_rank = rank_of[ic_];                                                          \
    aw_a = P.arrival ? arrival[ic_] : 0;                                             \
    aw_a = i_ < n ? aw_a : kNever;                                                   \
  } while (0)
    // the first word of the two-level bitmap with bits left, and its records
    // (loaded when the word changes)
#define SK_F_FIND()                                                                  \
  do {                                                                               \
    const uint64_t w1_ = L1[lane < nw1 ? lane : nw1 - 1];                            \
    const uint64_t nz_ = wave::ballot(w1_ != 0ull) & lane_span(0, nw1);              \
    f_word = 0ull;                                                                   \
    if (nz_ != 0ull) {                                                               \
      const int j1_ = __builtin_ctzll(nz_);                                          \
      const uint64_t w1v_ = wave::readlane_u64(w1_, j1_);                            \
      const int j0_ = j1_ * 64 + __builtin_ctzll(w1v_);                              \
      f_word = uniform_u64(L0[j0_]);                                                 \
      if (f_base != j0_ * 64) {                                                      \
        f_base = j0_ * 64;                                                           \
        /* (ranks past the last never wait: their lanes hold its record) */          \
        const int rr_ = f_base + lane < n ? f_base + lane : n - 1;                   \
        const uint64_t rv_ = rec[rr_];                                               \
        fw_key = static_cast<uint32_t>(rv_);                                         \
        fw_so = static_cast<uint32_t>(rv_ >> 32);                                    \
        if (kQueue) fw_u = upper_k[rr_];                                             \
      }                                                                              \
    }                                                                                \
  } while (0)
    // A_min: the first NP_ entries of the pending row join the sorted set.  An
    // entry takes the lane below its place and the smaller ones move down by one.
    // When the row has no lane left below, its upper part first goes to the stack
    // (if it is long) and the rest moves up by 32 lanes; an entry above the whole
    // row goes into the stack when that is not empty, below the smaller entries
    // there (they move up by one slot, 64 at a time).  No room: `status` says so.
#define SK_V_INSERT(NP_)                                                             \
  for (int q_ = 0; q_ < (NP_); ++q_) {                                               \
    const uint32_t ik_ = wave::readlane_u(pn_key, q_), is_ = wave::readlane_u(pn_so, q_); \
    int p_ = __builtin_popcountll(wave::ballot(vw_key < ik_));                       \
    if (SK_RARE(v_lo == 0)) {                                                        \
      if (v_hi > 32) {                                                               \
        if (v_sp + v_hi - 24 > cap_v - n_ovf) {                                      \
          status = P.retry_v_status;                                                 \
          q_ = (NP_);                                                                \
          continue;                                                                  \
        }                                                                            \
        v_store(lane_span(24, v_hi), v_sp + v_hi - 1 - lane, (static_cast<uint64_t>(vw_so) << 32) | vw_key); \
        v_sp += v_hi - 24;                                                           \
        v_hi = 24;                                                                   \
      }                                                                              \
      const int from_ = (lane ^ 32) << 2;                                            \
      const uint32_t mk_ = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from_, static_cast<int32_t>(vw_key))); \
      vw_so = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from_, static_cast<int32_t>(vw_so))); \
      vw_key = lane < 32 ? 0u : lane < 32 + v_hi ? mk_ : 0xFFFFFFFFu;                \
      v_lo = 32;                                                                     \
      v_hi += 32;                                                                    \
      p_ = __builtin_popcountll(wave::ballot(vw_key < ik_));                         \
    }                                                                                \
    if (SK_RARE(p_ == v_hi && v_sp > 0)) {                                           \
      if (v_sp + 1 > cap_v - n_ovf) {                                                \
        status = P.retry_v_status;                                                   \
        q_ = (NP_);                                                                  \
        continue;                                                                    \
      }                                                                              \
      int moved_ = 0;                                                                \
      for (;;) {                                                                     \
        const int ix_ = v_sp - 1 - moved_ - lane;                                    \
        const uint64_t e_ = v_load(ix_ >= 0 ? ix_ : 0);                              \
        const uint64_t less_ = wave::ballot(ix_ >= 0 && static_cast<uint32_t>(e_) < ik_); \
        const int c_ = __builtin_popcountll(less_);                                  \
        v_store(less_, ix_ + 1, e_);                                                 \
        moved_ += c_;                                                                \
        if (c_ < 64) break;                                                          \
      }                                                                              \
      v_store(1ull, v_sp - moved_, (static_cast<uint64_t>(is_) << 32) | ik_);        \
      ++v_sp;                                                                        \
    } else {                                                                         \
      --p_;                                                                          \
      const uint32_t dk_ = static_cast<uint32_t>(wave::dpp<wave::kDppWaveShl1>(static_cast<int32_t>(vw_key))); \
      const uint32_t ds_ = static_cast<uint32_t>(wave::dpp<wave::kDppWaveShl1>(static_cast<int32_t>(vw_so)));  \
      vw_key = lane < p_ ? dk_ : vw_key;                                             \
      vw_so = lane < p_ ? ds_ : vw_so;                                               \
      vw_key = wave::writelane_u(vw_key, ik_, p_);                                   \
      vw_so = wave::writelane_u(vw_so, is_, p_);                                     \
      --v_lo;                                                                        \
    }                                                                                \
  }
    // A_l: the register row moves to the queue's head when the head leaves it
#define SK_Q_WINDOW()                                                                \
  do {                                                                               \
    if (q_n > 0 && (q_head - q_base >= 64 || q_head < q_base)) {                     \
      wave::wait_stores();                                                           \
      q_base = q_head;                                                               \
      const int j_ = q_head + lane < n ? q_head + lane : n - 1;                      \
      const uint64_t w_ = static_cast<uint64_t>(qg[j_]);                             \
      vw_key = (static_cast<uint32_t>(w_ >> 48) << kIdxBits) | (static_cast<uint32_t>(w_) & kIdxMask); \
      vw_so = (static_cast<uint32_t>(w_ >> 17) & 0xFFFFu) | ((static_cast<uint32_t>(w_ >> 33) & 0x7FFFu) << 16); \
    }                                                                                \
  } while (0)
    // BODY with the compile-time row index r equal to the uniform row RR_
#define SK_AT_ROW(RR_, BODY)                                                         \
  _Pragma("unroll") for (int r = 0; r < ROWS; ++r) {                                 \
    if (r == (RR_)) {                                                                \
      BODY                                                                           \
    }                                                                                \
  }
    // A run with planned end EK_ and x = XK_ leaves: every run with
    // t+1 < r_end <= EK_ loses its share of f at its own planned end.
#define SK_DROP_SHARE(XK_, EK_)                                                      \
  do {                                                                               \
    const uint32_t lo_ = static_cast<uint32_t>(t) + 2u;                              \
    const int32_t w_ = (EK_) - (t + 1);                                              \
    const uint32_t span_ = w_ > 0 ? static_cast<uint32_t>(w_) : 0u;                  \
    const int32_t dx_ = t_r - (XK_);                                                 \
    _Pragma("unroll") for (int r_ = 0; r_ < ROWS; ++r_) {                            \
      const bool in_ = static_cast<uint32_t>(r_end[r_]) - lo_ < span_;               \
      r_f[r_] = in_ ? r_f[r_] - r_end[r_] + dx_ : r_f[r_];                           \
    }                                                                                \
  } while (0)

    // Issue priority among the waves of a SIMD: the more requests an instance
    // still has to complete, the higher (four levels by the unfinished
    // fraction), so the instances that bound the launch are not slowed by
    // their SIMD-mates; where a batch mixes interval widths (A_min with upper
    // bounds), the static class of the instance and whether half of it is
    // done instead (PRIO false: none).  Outputs do not depend on it.
    // (CLS false: an instance of the code without the class read, for the
    // launches that never have classes.)  The level changes when n_done reaches
    // prio_next.
    const int pcls = CLS ? ((kAmin && P.pclass) ? P.pclass[k] : -1) : -1;
    int32_t prio_next = 0;
#define SK_SET_PRIORITY()                                                            \
  do {                                                                               \
    if (PRIO && SK_RARE(n_done >= prio_next)) {                                      \
      const int left_ = n - n_done;                                                  \
      int lv_;                                                                       \
      if (pcls >= 0) {                                                               \
        lv_ = pcls + (2 * left_ > n ? 1 : 0);                                        \
        prio_next = 2 * left_ > n ? (n + 1) / 2 : n + 1;                             \
      } else {                                                                       \
        lv_ = 4 * left_ > 3 * n ? 3 : 2 * left_ > n ? 2 : 4 * left_ > n ? 1 : 0;     \
        prio_next = lv_ > 0 ? n - lv_ * n / 4 : n + 1;                               \
      }                                                                              \
      if (lv_ >= 3) __builtin_amdgcn_s_setprio(3);                                   \
      else if (lv_ == 2) __builtin_amdgcn_s_setprio(2);                              \
      else if (lv_ == 1) __builtin_amdgcn_s_setprio(1);                              \
      else __builtin_amdgcn_s_setprio(0);                                            \
    }                                                                                \
  } while (0)
    SK_SET_PRIORITY();
    // the state at the admissions of step t, for the body with NR_ rows
#define SK_SAVE_STATE(NR_)                                                             \
  do {                                                                                 \
    _Pragma("unroll") for (int r = 0; r < kStateRows; ++r) {                           \
      const bool have = r < ROWS;                                                      \
      st->r_end[r] = have ? r_end[r < ROWS ? r : 0] : kEmpty;                          \
      st->r_x[r] = have ? r_x[r < ROWS ? r : 0] : 0;                                   \
      st->r_c[r] = have ? r_c[r < ROWS ? r : 0] : kNever;                              \
      st->r_f[r] = have ? r_f[r < ROWS ? r : 0] : 0;                                   \
      st->r_key[r] = have ? r_key[r < ROWS ? r : 0] : 0xFFFFFFFFu;                     \
      st->r_u[r] = have ? r_u[r < ROWS ? r : 0] : 0;                                   \
    }                                                                                  \
    st->fr_row = fr_row; st->fr_mask = fr_mask; st->N = N; st->X = X; st->t_r = t_r;   \
    st->next_c = next_c; st->aw_base = aw_base; st->aw_a = aw_a; st->aw_rank = aw_rank; \
    st->arr_ptr = arr_ptr; st->next_a = next_a; st->f_base = f_base; st->f_word = f_word; \
    st->fw_key = fw_key; st->fw_so = fw_so; st->n_done = n_done; st->retry_at = retry_at; \
    st->t = t; st->DT = DT; st->rsteps = rsteps; st->tot_ev = tot_ev;                  \
    st->next_rows = (NR_); st->resume = true;                                          \
    if constexpr (kAmin || kQueue) {                                                   \
      st->vw_key = vw_key; st->vw_so = vw_so;                                          \
    }                                                                                  \
    if constexpr (kAmin) {                                                             \
      st->pn_key = pn_key; st->pn_so = pn_so; st->v_lo = v_lo; st->v_hi = v_hi;        \
      st->v_sp = v_sp; st->n_pend = n_pend; st->n_ovf = n_ovf;                         \
    }                                                                                  \
    if constexpr (kSorted) {                                                           \
      st->e_max = e_max; st->f_max = f_max;                                            \
    }                                                                                  \
    if constexpr (kQueue) {                                                            \
      st->fw_u = fw_u; st->q_head = q_head; st->q_n = q_n; st->q_base = q_base;        \
    }                                                                                  \
  } while (0)
    // One loop for all of it, an iteration being the events of a step (kStep),
    // the start of its admissions (kAdmit) or its next candidate (kNext): with a
    // loop for the candidates inside the loop over the steps, every way out of
    // the inner one but the first would cost a flag to set and to test again,
    // since the compiler gives every loop one exit.
    constexpr int kStep = 0, kAdmit = 1, kNext = 2;
    int mode = FROM_STATE && st->resume ? kAdmit : kStep;
    int32_t wait_until = kNever, Pm = 0;
    // the batch of candidates: lanes of a register row (fromF: of fw_key and
    // fw_so, else of vw_key and vw_so), and f at the planned ends of four of
    // them, the next one's and those after it: candidate q's in lane 16 q of gf,
    // its end in ge (q_at = 16 q; 64: to be found)
    uint64_t rest = 0ull;
    bool fromF = true;
    int32_t ge = 0, gf = 0;
    int q_at = 64;
    for (;;) {
      if (mode != kNext) {
      if (mode == kStep) {
      if (SK_RARE(t > cap)) {
        status = SCHED_E_STEP_CAP;
        goto ended;
      }
      if (SK_RARE(t - t_r >= kRebase)) {
        const int32_t d = t - t_r;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) r_x[r] = static_cast<int32_t>(static_cast<uint32_t>(r_x[r]) + static_cast<uint32_t>(d));
        X += N * d;
        t_r = t;
      }
      // ---- 1. arrivals; requests cancelled at the previous step become eligible
      if (SK_RARE(t >= next_a)) {
        const int32_t head = f_word != 0ull ? f_base + __builtin_ctzll(f_word) : -1;
        // the cached word goes back to LDS before arrivals set bits in it
        if (f_word != 0ull) wave::lds_store64(1ull, l0_at + 8u * static_cast<uint32_t>(f_base >> 6), f_word);
        while (arr_ptr < n) {
          if (arr_ptr >= aw_base + 64) SK_LOAD_ARRIVALS();
          const uint64_t m = wave::ballot((aw_base + lane >= arr_ptr) && aw_a <= t);
          if (m == 0ull) break;
          wave::lds_or64(m, l0_at + 8u * static_cast<uint32_t>(aw_rank >> 6), 1ull << (aw_rank & 63));
          wave::lds_or64(m, l1_at + 8u * static_cast<uint32_t>(aw_rank >> 12), 1ull << ((aw_rank >> 6) & 63));
          arr_ptr += __builtin_popcountll(m);
          if (arr_ptr < aw_base + 64) break;
        }
        if (arr_ptr < n) {
          if (arr_ptr >= aw_base + 64) SK_LOAD_ARRIVALS();
          next_a = wave::readlane(aw_a, arr_ptr - aw_base);
        } else {
          next_a = wave::in_sgpr(kNever);
        }
        SK_F_FIND();
        if (head != f_base + __builtin_ctzll(f_word | (1ull << 63))) retry_at = wave::in_sgpr(0);
      }
      if (kAmin && n_pend > 0) {
        SK_V_INSERT(n_pend);
        while (SK_RARE(n_ovf > 0 && status == SCHED_OK)) {
          // up to 64 more from the last slots of the stack's array
          const int c = n_ovf < 64 ? n_ovf : 64;
          const uint64_t e = v_load(cap_v - n_ovf + (lane < c ? lane : 0));
          pn_key = static_cast<uint32_t>(e);
          pn_so = static_cast<uint32_t>(e >> 32);
          n_ovf -= c;
          SK_V_INSERT(c);
        }
        if (SK_RARE(status != SCHED_OK)) goto ended;
        n_pend = 0;
        retry_at = wave::in_sgpr(0);
      }

      // ---- 2. completions up to t (the policies whose runs all end as planned
      // may have passed several steps with completions, see the jump below); DT =
      // memory the runs that complete at t still hold (s + o each)
      DT = wave::in_sgpr(0);
      {
      bool stale_c = false;           // next_c has to be found again
      if (t >= next_c) {
        int32_t sx = 0, sd = 0, sl = 0;
        int ndone = 0;
        uint64_t at = 0ull;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          const bool hit = kOnPlan ? r_c[r] <= t : r_c[r] == t;
          const uint64_t m = wave::ballot(hit);
          if (m) {
            at = m;
            ndone += __builtin_popcountll(m);
            if (kEarly) {
              // planned with u >= o: the run may end before its planned end
              uint64_t mm = m;
              while (mm) {
                const int ln = __builtin_ctzll(mm);
                mm &= mm - 1;
                const int32_t ek = wave::readlane(r_end[r], ln);
                const int32_t xk = wave::readlane(r_x[r], ln);
                if (kSorted && ek == e_max) f_max -= xk - t_r + ek;
                if (ek > t + 1) {
                  SK_DROP_SHARE(xk, ek);
                  retry_at = wave::in_sgpr(0);
                }
              }
            }
            const uint32_t id = r_key[r] & kIdxMask;
            if (stage_c) wave::lds_store32(m, lc_at + 4u * id, static_cast<uint32_t>(kOnPlan ? r_c[r] : t));
            else wave::global_store32(m, cdst + id, static_cast<uint32_t>(kOnPlan ? r_c[r] : t));
            sx += hit ? r_x[r] : 0;
            if (kOnPlan) {
              sd += r_c[r] == t ? r_x[r] + (t - t_r) : 0;
              sl += hit ? t - r_c[r] : 0;
            }
            r_end[r] = hit ? kEmpty : r_end[r];
            r_c[r] = hit ? kNever : r_c[r];
            r_key[r] = hit ? 0xFFFFFFFFu : r_key[r];
            if (r == fr_row) fr_mask |= m;
          }
        }
        if (SK_USUAL(ndone > 0)) {
          // (the sums are that run's values in its lane when one run completes)
          int32_t sxw;
          if (kOnPlan) {
            int32_t late;
            if (ndone == 1) {
              const int ln = __builtin_ctzll(at);
              sxw = wave::readlane(sx, ln);
              DT = wave::readlane(sd, ln);
              late = wave::readlane(sl, ln);
            } else {
              const int32_t s4 = wave::sum4_i32(sx, sd, sl, 0);
              sxw = wave::readlane(s4, 0);
              DT = wave::readlane(s4, 16);
              late = wave::readlane(s4, 32);
            }
            rsteps -= late;  // (counted to t by the jump)
          } else {
            sxw = ndone == 1 ? wave::readlane(sx, __builtin_ctzll(at)) : wave::sum_i32(sx);
            DT = sxw + ndone * (t - t_r);
          }
          X -= sxw;
          N -= ndone;
          n_done += ndone;
          SK_SET_PRIORITY();
        }
        // ---- 3. done?
        if (SK_RARE(n_done == n)) goto ended;
        // ---- 3'. A_l: a run still present at its planned end t (planned with
        // l, so o > l) is promoted: it leaves, plans with u and joins the back of
        // the queue, lowest index first among this step's promotions
        if (kQueue) {
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
            if (wave::ballot(best != 0xFFFFFFFFu) == 0ull) break;
            const uint32_t iv = wave::min_u32_all(best);
            const uint64_t pm = wave::ballot(best == iv);
            const uint32_t imin = wave::uniform_u(iv);
            const int ln = __builtin_ctzll(pm);
            const int rr = wave::readlane(brow, ln);
            int32_t xk = 0, ck = 0, uk = 0;
            uint32_t kk = 0;
            SK_AT_ROW(rr, xk = wave::readlane(r_x[r], ln); ck = wave::readlane(r_c[r], ln);
                      uk = wave::readlane(r_u[r], ln); kk = wave::readlane_u(r_key[r], ln);
                      r_end[r] = wave::writelane(r_end[r], kEmpty, ln);
                      r_c[r] = wave::writelane(r_c[r], kNever, ln);
                      r_key[r] = wave::writelane_u(r_key[r], 0xFFFFFFFFu, ln);)
            if (rr == fr_row) fr_mask |= 1ull << ln;
            // its planned end is t itself: no later planned end loses a share
            X -= xk;
            N -= 1;
            const int32_t pk = t - static_cast<int32_t>(kk >> kIdxBits);
            const uint32_t sk = static_cast<uint32_t>(xk - t_r + pk);
            const uint32_t okk = static_cast<uint32_t>(ck - pk);
            const int slot = q_head + q_n;  // < n: each request is promoted at most once
            wave::global_store64(1ull, P.vglob + b + slot,
                                 imin | (static_cast<uint64_t>(sk) << 17) | (static_cast<uint64_t>(okk) << 33) |
                                     (static_cast<uint64_t>(uk) << 48));
            if (P.evictions) wave::global_add32(1ull, ev_at + imin, 1u);
            if (slot >= q_base && slot - q_base < 64) {
              vw_key = wave::writelane_u(vw_key, (static_cast<uint32_t>(uk) << kIdxBits) | imin, slot - q_base);
              vw_so = wave::writelane_u(vw_so, sk | (okk << 16), slot - q_base);
            }
            ++q_n;
            ++tot_ev;
          }
        }
        stale_c = true;
      }

      // ---- 4. A_min: cancel in ascending (o~, index) while memory at t+1 > M
      if (kAmin) {
        Pm = X + N * (t + 1 - t_r);
        if (Pm > M) {
          // which: the runs with the smallest keys until the rest fits (k_next:
          // one above the last key taken; the others' keys less k_next, the taken
          // ones' wrapping round to the top)
          uint32_t k_next = 0u;
          do {
            uint32_t best = r_key[0] - k_next;
#pragma unroll
            for (int r = 1; r < ROWS; ++r) {
              const uint32_t kk = r_key[r] - k_next;
              best = kk < best ? kk : best;
            }
            const uint32_t kmin = wave::min_u32(best) + k_next;
            // keys differ, so one slot matches
            uint64_t at = 0ull;
            int32_t xs = 0;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              const bool hit = r_key[r] == kmin;
              at |= wave::ballot(hit);
              xs = hit ? r_x[r] : xs;
            }
            const int32_t xk = wave::readlane(xs, __builtin_ctzll(at));
            X -= xk;
            N -= 1;
            Pm -= xk + t + 1 - t_r;
            k_next = kmin + 1u;
            // (no run left means no memory held)
          } while (Pm > M && N > 0);
          // then all of them at once: out of their slots, with what they would
          // plan with, into the pending row, startable from the next step
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            uint64_t cm = wave::ballot(r_key[r] < k_next);
            if (cm == 0ull) continue;
            const int c = __builtin_popcountll(cm);
            if (SK_RARE(n_pend + c > 64)) {
              // the pending row first goes to the last free slots of the stack's array
              if (v_sp + n_ovf + n_pend > cap_v) {
                status = P.retry_v_status;
                break;
              }
              n_ovf += n_pend;
              v_store(lane_span(0, n_pend), cap_v - n_ovf + lane, (static_cast<uint64_t>(pn_so) << 32) | pn_key);
              if (P.evictions) wave::global_add32(lane_span(0, n_pend), ev_at + (pn_key & kIdxMask), 1u);
              tot_ev += n_pend;
              n_pend = 0;
            }
            const bool gone = r_key[r] < k_next;
            const int32_t oh = static_cast<int32_t>(r_key[r] >> kIdxBits);
            const int32_t pk = r_end[r] - oh;
            const int32_t gen = t - pk;
            const int32_t nh = gen > oh ? gen : oh;
            const uint32_t nkey = (static_cast<uint32_t>(nh) << kIdxBits) | (r_key[r] & kIdxMask);
            const uint32_t so = static_cast<uint32_t>(r_x[r] - t_r + pk) | (static_cast<uint32_t>(r_c[r] - pk) << 16);
            stale_c = stale_c || (wave::ballot(r_c[r] == next_c) & cm) != 0ull;
            uint64_t fm = wave::ballot(r_end[r] > t + 1) & cm;   // those with shares ahead
            if (r == fr_row) fr_mask |= cm;
            do {
              const int ln = __builtin_ctzll(cm);
              cm &= cm - 1ull;
              pn_key = wave::writelane_u(pn_key, wave::readlane_u(nkey, ln), n_pend);
              pn_so = wave::writelane_u(pn_so, wave::readlane_u(so, ln), n_pend);
              ++n_pend;
            } while (cm != 0ull);
            while (fm != 0ull) {
              const int ln = __builtin_ctzll(fm);
              fm &= fm - 1ull;
              SK_DROP_SHARE(wave::readlane(r_x[r], ln), wave::readlane(r_end[r], ln));
            }
            r_end[r] = gone ? kEmpty : r_end[r];
            r_c[r] = gone ? kNever : r_c[r];
            r_key[r] = gone ? 0xFFFFFFFFu : r_key[r];
          }
          if (SK_RARE(status != SCHED_OK)) goto ended;
          // the cancellation counts of the step's pending requests at once
          if (P.evictions) wave::global_add32(lane_span(0, n_pend), ev_at + (pn_key & kIdxMask), 1u);
          tot_ev += n_pend;
          retry_at = wave::in_sgpr(0);
        }
      }
      if (stale_c) {
        // next event: a completion (A_l: or a planned end, where a run is
        // promoted); empty slots read as unsigned are above every step
        uint32_t cmin = 0xFFFFFFFFu;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          uint32_t ev = static_cast<uint32_t>(r_c[r]);
          if (kQueue) {
            const uint32_t pe = static_cast<uint32_t>(r_end[r]);
            ev = pe < ev ? pe : ev;
          }
          cmin = ev < cmin ? ev : cmin;
        }
        next_c = static_cast<int32_t>(wave::min_u32(cmin));  // kNever when nothing runs
      }
      }

      // ---- shrink: once the runs fit a smaller body with room to spare, move
      // the runs of the upper rows into free slots of the lower ones (the
      // order of slots never matters: every choice is by key) and hand over
      if constexpr (TO_STATE && ROWS > 2) {
        int target = 0;
        if (N <= 64 * 2 - kShrinkSpare) target = 2;
        else if (ROWS > 3 && N <= 64 * 3 - kShrinkSpare) target = 3;
        else if (ROWS > 5 && N <= 64 * 5 - kShrinkSpare) target = 5;
        else if (ROWS > 8 && N <= 64 * 8 - kShrinkSpare) target = 8;
        else if (ROWS > 10 && N <= 64 * 10 - kShrinkSpare) target = 10;
        else if (ROWS > 12 && N <= 64 * 12 - kShrinkSpare) target = 12;
        if (SK_RARE(target > 0)) {
          uint64_t fm[ROWS];
#pragma unroll
          for (int r = 0; r < ROWS; ++r) fm[r] = wave::ballot(r_end[r] == kEmpty);
#pragma unroll
          for (int h = ROWS - 1; h >= 2; --h) {
            if (h < target) break;
            uint64_t m = ~fm[h];
            while (m) {
              const int ln = __builtin_ctzll(m);
              m &= m - 1;
              // the lowest row below the target with a free lane
              int l = 0;
              uint64_t fl_mask = 0;
#pragma unroll
              for (int r = ROWS - 1; r >= 0; --r) {
                const bool ok = r < target && fm[r] != 0ull;
                l = ok ? r : l;
                fl_mask = ok ? fm[r] : fl_mask;
              }
              const int fl = __builtin_ctzll(fl_mask);
              const int32_t me = wave::readlane(r_end[h], ln), mx = wave::readlane(r_x[h], ln);
              const int32_t mc = wave::readlane(r_c[h], ln), mf = wave::readlane(r_f[h], ln);
              const int32_t mu = wave::readlane(r_u[h], ln);
              const uint32_t mk = wave::readlane_u(r_key[h], ln);
              SK_AT_ROW(l, r_end[r] = wave::writelane(r_end[r], me, fl); r_x[r] = wave::writelane(r_x[r], mx, fl);
                        r_c[r] = wave::writelane(r_c[r], mc, fl); r_f[r] = wave::writelane(r_f[r], mf, fl);
                        r_u[r] = wave::writelane(r_u[r], mu, fl); r_key[r] = wave::writelane_u(r_key[r], mk, fl);
                        fm[r] &= ~(1ull << fl);)
              r_end[h] = wave::writelane(r_end[h], kEmpty, ln);
              r_c[h] = wave::writelane(r_c[h], kNever, ln);
              r_key[h] = wave::writelane_u(r_key[h], 0xFFFFFFFFu, ln);
            }
          }
          fr_row = 0;
          fr_mask = 0ull;  // the next admission looks for a free row
          handoff = target;
          status = kResume;
          goto ended;
        }
      }

      }
      // ---- 5. admission of the longest feasible prefix in key order, one
      // candidate an iteration.  wait_until: the step before which the head
      // cannot start unless something else happens (kNever: it waits for that).
      wait_until = wave::in_sgpr(kNever);
      if (t < retry_at) {
        wait_until = retry_at;
        goto admitted;
      }
      Pm = X + N * (t + 1 - t_r);  // memory at t+1: every running request is present
      rest = 0ull;
      }
      if (rest == 0ull) {
        // the next batch: a run of fresh requests, or (A_min) of cancelled ones,
        // with no candidate of the other set between them (A_l: every fresh
        // request comes before the promoted ones)
        q_at = 64;
        if (SK_RARE(f_word == 0ull && f_base >= 0)) {
          // the word in scalar registers has been emptied: the next one
          const int j0 = f_base >> 6;
          wave::lds_store64(1ull, l0_at + 8u * static_cast<uint32_t>(j0), 0ull);
          wave::lds_and64(1ull, l1_at + 8u * static_cast<uint32_t>(j0 >> 6), ~(1ull << (j0 & 63)));
          SK_F_FIND();
          if (f_word == 0ull) f_base = -1;
        }
        rest = f_word;
        if constexpr (kAmin) {
          if (SK_RARE(v_lo == v_hi && v_sp > 0)) {
            // refill the register row from the top of the stack
            const int c = v_sp < 32 ? v_sp : 32;
            const int j = v_sp + 15 - lane;  // lane 16 gets the top
            const uint64_t e = v_load(j < 0 ? 0 : j < v_sp ? j : v_sp - 1);
            vw_key = lane < 16 ? 0u : lane < 16 + c ? static_cast<uint32_t>(e) : 0xFFFFFFFFu;
            vw_so = static_cast<uint32_t>(e >> 32);
            v_lo = 16;
            v_hi = 16 + c;
            v_sp -= c;
          }
          const uint32_t fk = f_word != 0ull ? wave::readlane_u(fw_key, __builtin_ctzll(f_word)) : 0xFFFFFFFFu;
          const uint32_t vk = v_lo < v_hi ? wave::readlane_u(vw_key, v_lo) : 0xFFFFFFFFu;
          fromF = fk <= vk;
          rest = fromF ? f_word & wave::ballot(fw_key < vk) : (~0ull << v_lo) & wave::ballot(vw_key < fk);
        }
        if constexpr (kQueue) {
          fromF = true;
          if (f_word == 0ull) {
            SK_Q_WINDOW();
            const int d = q_head - q_base;
            const int m = q_n < 64 - d ? q_n : 64 - d;
            rest = q_n > 0 ? lane_span(d, d + m) : 0ull;
            fromF = false;
          }
        }
        if (rest == 0ull) {
          // nothing waits
          if (kDrains && SK_RARE(next_a == kNever)) {
            // nor will anything: the runs end as they are.  A run that completes at
            // C <= cap counts at steps t to C - 1, another to the cap
            int32_t left = 0;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              const bool run = r_c[r] != kNever;
              const bool ends = run && r_c[r] <= cap;
              const uint64_t m = wave::ballot(ends);
              left += run && !ends ? 1 : 0;
              rsteps += wave::sum_i32(run ? (ends ? r_c[r] : cap + 1) - t : 0);
              if (stage_c) wave::lds_store32(m, lc_at + 4u * (r_key[r] & kIdxMask), static_cast<uint32_t>(r_c[r]));
              else wave::global_store32(m, cdst + (r_key[r] & kIdxMask), static_cast<uint32_t>(r_c[r]));
            }
            if (wave::ballot(left != 0) != 0ull) status = SCHED_E_STEP_CAP;
            goto ended;
          }
          wait_until = kOnPlan ? next_a : wave::in_sgpr(kNever);
          goto admitted;
        }
      }
      {
        const uint32_t bkey = (kAmin || kQueue) && !fromF ? vw_key : fw_key;
        const uint32_t bso = (kAmin || kQueue) && !fromF ? vw_so : fw_so;
        const int j = __builtin_ctzll(rest);
        const uint32_t c_so = wave::readlane_u(bso, j);
        const int32_t s = static_cast<int32_t>(c_so & 0xFFFFu);
        // step t + 1, and step t, at which runs completing at t hold s + o (the
        // latter is implied by the former when DT = 0)
        const int32_t at_t = Pm + (DT - N);
        if ((Pm + 1 > at_t ? Pm + 1 : at_t) + s > M) {
          wait_until = Pm + s + 1 > M ? wave::in_sgpr(kNever) : t + 1;
          goto admitted;
        }
        const uint32_t c_key = wave::readlane_u(bkey, j);
        const int32_t c_o = static_cast<int32_t>(c_so >> 16);
        const int32_t est = ALGO == SCHED_ARANDOM ? c_o : static_cast<int32_t>(c_key >> kIdxBits);
        const int32_t E = t + est;
        // the planned ends c in (t+1, E] gain its share s + c - t; none may
        // pass M (step t+1 was tested above), nor f at its own end E
        const uint32_t lo2 = static_cast<uint32_t>(t) + 2u;
        const uint32_t span = static_cast<uint32_t>(est - 1);
        const int32_t dh = s - t;
        int32_t nf[ROWS];
        int32_t fmx = 0;
        const bool top = kSorted && E >= e_max;   // no planned end is above E
        if (top) {
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            nf[r] = r_end[r] > t + 1 ? r_f[r] + r_end[r] + dh : r_f[r];
            fmx = nf[r] > fmx ? nf[r] : fmx;
          }
        } else {
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            const bool in = static_cast<uint32_t>(r_end[r]) - lo2 < span;
            nf[r] = in ? r_f[r] + r_end[r] + dh : r_f[r];
            fmx = nf[r] > fmx ? nf[r] : fmx;
          }
        }
        if (wave::ballot(fmx > M) != 0ull) {
          // each violating end improves by one per step, or leaves the window
          int32_t fix = 0;
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            const int32_t over = nf[r] - M, left = r_end[r] - 1 - t;
            const int32_t m = over < left ? over : left;
            fix = (over > 0 && m > fix) ? m : fix;
          }
          retry_at = t + wave::max_i32(fix);
          wait_until = retry_at;
          goto admitted;
        }
        int32_t fe;
        if (top) {
          fe = (E == e_max ? f_max : 0) + s + est;
          q_at = 64;
        } else {
          if (q_at == 64) {
            // planned length of each lane's candidate
            const int32_t lest =
                ALGO == SCHED_ARANDOM ? static_cast<int32_t>(bso >> 16) : static_cast<int32_t>(bkey >> kIdxBits);
            uint64_t g = rest & (rest - 1ull);
            int32_t e1 = kNever, e2 = kNever, e3 = kNever;
            if (g != 0ull) {
              e1 = t + wave::readlane(lest, __builtin_ctzll(g));
              g &= g - 1ull;
              if (g != 0ull) {
                e2 = t + wave::readlane(lest, __builtin_ctzll(g));
                g &= g - 1ull;
                if (g != 0ull) e3 = t + wave::readlane(lest, __builtin_ctzll(g));
              }
            }
            ge = wave::writelane(ge, e1, 16);
            ge = wave::writelane(ge, e2, 32);
            ge = wave::writelane(ge, e3, 48);
            int32_t fl0 = 0, fl1 = 0, fl2 = 0, fl3 = 0;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              fl0 = r_end[r] >= E ? fl0 + r_x[r] + (E - t_r) : fl0;
              fl1 = r_end[r] >= e1 ? fl1 + r_x[r] + (e1 - t_r) : fl1;
              fl2 = r_end[r] >= e2 ? fl2 + r_x[r] + (e2 - t_r) : fl2;
              fl3 = r_end[r] >= e3 ? fl3 + r_x[r] + (e3 - t_r) : fl3;
            }
            gf = wave::sum4_i32(fl0, fl1, fl2, fl3);
            q_at = 0;
            if (kGroup && !CAPPED && e3 != kNever && __builtin_popcountll(fr_mask) >= 4) {
              // The next three candidates with it, when their memory fits at t and
              // t + 1 and the free row has room: the shares of all four on every row
              // and on their own planned ends, and one test, which passes exactly
              // when each would pass after those before it (shares only add).  When
              // it does not pass, they are taken one by one, with the same sums.
              // (A_min: 4096 x 1000 in 8.2 ms instead of 9.1, 65536 x 2000 in 109
              // instead of 117; A_random 3000 x 1500 in 1.23 instead of 1.33; A_l
              // 1024 x 10000 in 23.4 instead of 25.2.  Groups of two to four were
              // slower than none on the last two.)
              const uint64_t rest1 = rest & (rest - 1ull), rest2 = rest1 & (rest1 - 1ull), rest3 = rest2 & (rest2 - 1ull);
              const int j1 = __builtin_ctzll(rest1), j2 = __builtin_ctzll(rest2), j3 = __builtin_ctzll(rest3);
              const uint32_t so1 = wave::readlane_u(bso, j1), so2 = wave::readlane_u(bso, j2), so3 = wave::readlane_u(bso, j3);
              const int32_t s1 = static_cast<int32_t>(so1 & 0xFFFFu), s2 = static_cast<int32_t>(so2 & 0xFFFFu);
              const int32_t s3 = static_cast<int32_t>(so3 & 0xFFFFu);
              const int32_t s4 = s + s1 + s2 + s3;
              // (a run adds one less at t than at t + 1)
              if ((Pm + 4 > at_t ? Pm + 4 : at_t) + s4 <= M) {
                const int32_t d1 = s1 - t, d2 = s2 - t, d3 = s3 - t;
                const uint32_t w1 = static_cast<uint32_t>(e1 - t - 1), w2 = static_cast<uint32_t>(e2 - t - 1);
                const uint32_t w3 = static_cast<uint32_t>(e3 - t - 1);
                int32_t gmx = 0;
                int32_t ng[ROWS];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                  const uint32_t c = static_cast<uint32_t>(r_end[r]) - lo2;
                  ng[r] = c < w1 ? nf[r] + r_end[r] + d1 : nf[r];
                  ng[r] = c < w2 ? ng[r] + r_end[r] + d2 : ng[r];
                  ng[r] = c < w3 ? ng[r] + r_end[r] + d3 : ng[r];
                  gmx = ng[r] > gmx ? ng[r] : gmx;
                }
                ge = wave::writelane(ge, E, 0);
                int32_t f4 = gf;
                f4 = ge <= E ? f4 + ge + dh : f4;
                f4 = ge <= e1 ? f4 + ge + d1 : f4;
                f4 = ge <= e2 ? f4 + ge + d2 : f4;
                f4 = ge <= e3 ? f4 + ge + d3 : f4;
                if ((wave::ballot(gmx > M) | (wave::ballot(f4 > M) & 0x0001000100010001ull)) == 0ull) {
#pragma unroll
                  for (int r = 0; r < ROWS; ++r) r_f[r] = ng[r];
                  const uint64_t m1 = fr_mask & (fr_mask - 1ull), m2 = m1 & (m1 - 1ull), m3 = m2 & (m2 - 1ull);
                  const int l0 = __builtin_ctzll(fr_mask), l1 = __builtin_ctzll(m1), l2 = __builtin_ctzll(m2);
                  const int l3 = __builtin_ctzll(m3);
                  const int32_t f0 = wave::readlane(f4, 0), f1 = wave::readlane(f4, 16);
                  const int32_t f2 = wave::readlane(f4, 32), f3 = wave::readlane(f4, 48);
                  const int32_t xb = t_r - t;
                  const int32_t o1 = static_cast<int32_t>(so1 >> 16), o2 = static_cast<int32_t>(so2 >> 16);
                  const int32_t o3 = static_cast<int32_t>(so3 >> 16);
                  const uint32_t k1 = wave::readlane_u(bkey, j1), k2 = wave::readlane_u(bkey, j2), k3 = wave::readlane_u(bkey, j3);
                  int32_t u0 = 0, u1 = 0, u2 = 0, u3 = 0;
                  if (kQueue) {
                    u0 = fromF ? wave::readlane(fw_u, j) : est;
                    u1 = fromF ? wave::readlane(fw_u, j1) : e1 - t;
                    u2 = fromF ? wave::readlane(fw_u, j2) : e2 - t;
                    u3 = fromF ? wave::readlane(fw_u, j3) : e3 - t;
                  }
#define SK_PUT(LN_, E_, S_, O_, K_, F_, U_)                                          \
  r_end[r] = wave::writelane(r_end[r], E_, LN_);                                     \
  r_x[r] = wave::writelane(r_x[r], xb + S_, LN_);                                    \
  r_c[r] = wave::writelane(r_c[r], t + O_, LN_);                                     \
  r_key[r] = wave::writelane_u(r_key[r], K_, LN_);                                   \
  r_f[r] = wave::writelane(r_f[r], F_, LN_);                                         \
  if (kQueue) r_u[r] = wave::writelane(r_u[r], U_, LN_);
                  SK_AT_ROW(fr_row, SK_PUT(l0, E, s, c_o, c_key, f0, u0) SK_PUT(l1, e1, s1, o1, k1, f1, u1)
                            SK_PUT(l2, e2, s2, o2, k2, f2, u2) SK_PUT(l3, e3, s3, o3, k3, f3, u3))
#undef SK_PUT
                  fr_mask = m3 & (m3 - 1ull);
                  int32_t near = c_o < o1 ? c_o : o1;
                  near = o2 < near ? o2 : near;
                  near = o3 < near ? o3 : near;
                  if (kQueue) {
                    near = est < near ? est : near;
                    near = e1 - t < near ? e1 - t : near;
                    near = e2 - t < near ? e2 - t : near;
                    near = e3 - t < near ? e3 - t : near;
                  }
                  next_c = t + near < next_c ? t + near : next_c;
                  X += s4 + 4 * xb;
                  N += 4;
                  Pm += s4 + 4;
                  rest = rest3 & (rest3 - 1ull);
                  if (kAmin && !fromF) {
                    v_lo += 4;
                    vw_key = lane < v_lo ? 0u : vw_key;
                  } else if (kQueue && !fromF) {
                    q_head += 4;
                    q_n -= 4;
                  } else {
                    f_word &= ~1ull << j3;
                  }
                  retry_at = wave::in_sgpr(0);
                  q_at = 64;
                  mode = kNext;
                  continue;
                }
              }
            }
          }
          fe = wave::readlane(gf, q_at) + s + est;
        }
        if (SK_RARE(est > 1 && fe > M)) {
          // f at the sliding end only grows until it passes the next planned end
          int32_t emin = kNever;
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
            const int32_t e = r_end[r];
            emin = (e >= E && e < emin) ? e : emin;
          }
          retry_at = static_cast<int32_t>(wave::min_u32(static_cast<uint32_t>(emin))) - est + 1;
          wait_until = retry_at;
          goto admitted;
        }
        // admit: start at p = t, in a free slot (without one nothing has
        // changed for this candidate)
        if (CAPPED && SK_RARE(N >= P.run_cap)) {
          status = retry_status;
          goto ended;
        }
        if (SK_RARE(fr_mask == 0ull)) {
          int rr = -1;
          uint64_t mm = 0ull;
#pragma unroll
          for (int r = ROWS - 1; r >= 0; --r) {
            const uint64_t m = wave::ballot(r_end[r] == kEmpty);
            rr = m ? r : rr;
            mm = m ? m : mm;
          }
          if (SK_RARE(rr < 0)) {
            // hand the state at this admission to the body above, if there is one
            handoff = TO_STATE ? ladder_up(ROWS, kStateRows) : 0;
            status = handoff > 0 ? kResume : retry_status;
            goto ended;
          }
          fr_row = rr;
          fr_mask = mm;
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) r_f[r] = nf[r];
        {
          const int32_t xw = t_r - t + s;
          const int32_t cw = t + c_o;
          const int ln = __builtin_ctzll(fr_mask);
          fr_mask &= fr_mask - 1;
          const int32_t uw = !kQueue ? 0 : fromF ? wave::readlane(fw_u, j) : est;
          SK_AT_ROW(fr_row, r_end[r] = wave::writelane(r_end[r], E, ln); r_x[r] = wave::writelane(r_x[r], xw, ln);
                    r_c[r] = wave::writelane(r_c[r], cw, ln); r_key[r] = wave::writelane_u(r_key[r], c_key, ln);
                    r_f[r] = wave::writelane(r_f[r], fe, ln);
                    if (kQueue) r_u[r] = wave::writelane(r_u[r], uw, ln);)
          const int32_t ew = kQueue && E < cw ? E : cw;  // A_l: promotion at E
          next_c = ew < next_c ? ew : next_c;
          X += xw;
        }
        if (kSorted && top) {
          e_max = E;
          f_max = fe;
        } else {
          // the later candidates of the four whose end it reaches
          gf = ge <= E ? gf + ge + dh : gf;
          q_at += 16;
        }
        N += 1;
        Pm += s + 1;
        rest &= rest - 1ull;
        if (kAmin && !fromF) {
          vw_key = wave::writelane_u(vw_key, 0u, j);
          ++v_lo;
        } else if (kQueue && !fromF) {
          ++q_head;
          --q_n;
        } else {
          f_word &= f_word - 1ull;
        }
        retry_at = wave::in_sgpr(0);
        mode = kNext;
        continue;
      }

    admitted:
      // ---- 6. this step processes every running request once
      rsteps += N;
      {
      int32_t tn = t + 1;
      if (!kAmin || n_pend == 0) {
        // Nothing changes before the next completion, arrival or (A_min)
        // overflow; until then the head cannot start before wait_until.  Where
        // every run ends as planned, completions change nothing for a head that
        // waits for planned ends to pass (f keeps its values), so the jump goes
        // past them; the steps they no longer run are taken off when they are
        // processed.
        int32_t jump = wait_until;
        if (!(kOnPlan && wait_until <= cap)) jump = next_c < jump ? next_c : jump;
        jump = wave::in_sgpr(next_a < jump ? next_a : jump);
        const int32_t lim = t_r + kRebase;
        jump = wave::in_sgpr(lim < jump ? lim : jump);
        jump = cap + 1 < jump ? cap + 1 : jump;
        if (kAmin && N > 0) {
          // first step whose projection exceeds M, if it comes before the jump
          // (jump - t <= 2^16 and N <= 2^10 here, and Pm <= M < 2^30)
          Pm = X + N * (t + 1 - t_r);
          if (Pm + N * (jump - 1 - t) > M) {
            // (M - Pm) / N, below 2^16: the float quotient is off by at most one
            const int32_t d = M - Pm;
            int32_t qd = wave::uniform(static_cast<int32_t>(static_cast<float>(d) * __builtin_amdgcn_rcpf(static_cast<float>(N))));
            const int32_t rem = d - qd * N;
            qd += rem < 0 ? -1 : rem >= N ? 1 : 0;
            const int32_t tev = t + qd + 1;
            jump = tev < jump ? tev : jump;
          }
        }
        if (jump > tn) {
          rsteps += static_cast<int64_t>(N) * (jump - tn);
          tn = jump;
        }
      }
      t = tn;
      mode = kStep;
      }
    }
  ended:
    if constexpr (TO_STATE) {
      // every way out of a handing-over body writes the whole state (so that the
      // state a body started from is dead while it runs)
      SK_SAVE_STATE(handoff);
    } else {
      st->rsteps = rsteps;
      st->tot_ev = tot_ev;
    }
  }
  return status;
}
// The end of an instance's simulation: its totals from the per-request outputs
// (with tie keys, these are first copied from the staging arrays, by id, to the
// outputs, by index).  st0, status: before and after; vglobal: whether the
// launch keeps no cancelled set in LDS.  Outside of the bodies, so that a ladder
// kernel holds it once and its bodies' loops hold no branch on the lane.
__device__ __forceinline__ void finish_instance(const Params& P, const int k, const int st0, const int status,
                                                int64_t rsteps, int64_t tot_ev, const bool vglobal) {
  extern __shared__ uint64_t lds64[];
  const int lane = static_cast<int>(threadIdx.x);
  const int64_t b = P.offsets[k];
  const int n = st0 == SCHED_OK ? static_cast<int>(P.offsets[k + 1] - b) : 0;
  wave::wait_stores();
  __syncthreads();
  const bool keep = (status == SCHED_OK || status == SCHED_E_STEP_CAP) && n > 0;
  const bool tie = P.tie_key != nullptr;
  const bool st_c = P.stage_comp != 0;
  int64_t tel = 0, mk = 0;
  if (keep) {
    const int32_t* lc = reinterpret_cast<const int32_t*>(lds64 + P.nw_max + P.nw1_max + (vglobal ? 0 : P.cap_v));
    for (int c = 0; c < n; c += 64) {
      const int i = c + lane;
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
    for (int c = 0; c < n; c += 64) {
      const int i = c + lane;
      if (i < n) {
        comp[b + i] = -1;
        if (P.evictions) evs[b + i] = 0;
      }
    }
  }
  tel = wave::sum_i64(tel);
  mk = wave::max_i64(mk);
  if (!keep) {
    rsteps = 0;
    tot_ev = 0;
  }
  if (lane == 0) {
    P.total_latency[k] = tel;
    if (P.makespan) P.makespan[k] = static_cast<int32_t>(mk);
    if (P.request_steps) P.request_steps[k] = rsteps;
    if (P.total_evictions) P.total_evictions[k] = tot_ev;
    P.status[k] = status;
  }
}
#undef SK_SET_PRIORITY
#undef SK_RARE
#undef SK_USUAL
#undef SK_SAVE_STATE
#undef SK_LOAD_ARRIVALS
#undef SK_F_FIND
#undef SK_V_INSERT
#undef SK_Q_WINDOW
#undef SK_AT_ROW
#undef SK_DROP_SHARE

// One wave per instance.  RETRY_PASS: only instances handed over by an
// earlier launch for a reason this pass takes (P.run_mask) run, held to
// P.run_cap runs at once.
template <int ALGO, int ROWS, bool RETRY_PASS, bool VGLOBAL = false>
__global__ __launch_bounds__(64) void k_simulate(Params P) {
  const int k = blockIdx.x;
  if (P.algo_of && P.algo_of[k] != ALGO) return;  // adaptive run: the other policy's instance
  int st0 = P.status[k];
  if (RETRY_PASS) {
    const bool take = (st0 == kRetryRows && (P.run_mask & 1)) || (st0 == kRetryV && (P.run_mask & 2));
    if (!take) return;
    st0 = SCHED_OK;
  }
  WaveState st;
  st.rsteps = 0;
  st.tot_ev = 0;
  const int status = wave_instance<ALGO, ROWS, false, false, VGLOBAL, RETRY_PASS>(P, k, st0, P.retry_status, &st);
  finish_instance(P, k, st0, status, st.rsteps, st.tot_ev, VGLOBAL);
}

// One wave per instance on the row ladder: the simulation starts with 2
// register rows and moves, state and all, to the body with 3, 5, 8 or 10 rows
// (the wide ladder, below: also 12 and 16) as its running set grows and back down
// as it shrinks, so that every scan covers about as many rows as the instance has
// runs (most of an instance's events happen with at most 128 runs).
template <int ALGO>
__device__ __forceinline__ void wide_ladder_instance(const Params& P, const int k) {
  if (P.algo_of && P.algo_of[k] != ALGO) return;
  int st0 = P.status[k];
  if (P.run_mask) {
    // a retry pass: only the instances an earlier pass handed over
    const bool take = (st0 == kRetryRows && (P.run_mask & 1)) || (st0 == kRetryV && (P.run_mask & 2));
    if (!take) return;
    st0 = SCHED_OK;
  }
  int arr_ptr = 0;
  if (st0 == SCHED_OK) {
    // the bodies all resume from a state, so the bitmaps and staged outputs
    // are set up here
    extern __shared__ uint64_t lds64[];
    const int64_t b = P.offsets[k];
    const int n = static_cast<int>(P.offsets[k + 1] - b);
    arr_ptr = start_waiting(P, b, n, lds64, lds64 + P.nw_max);
    int32_t* lc = reinterpret_cast<int32_t*>(lds64 + P.nw_max + P.nw1_max + P.cap_v);
    if (P.stage_comp)
      for (int i = threadIdx.x; i < n; i += 64) lc[i] = -1;
    __syncthreads();
  }
  const bool empty = st0 == SCHED_OK && P.offsets[k + 1] == P.offsets[k];
  if (st0 != SCHED_OK || empty) {
    // nothing to simulate: zero totals (the per-request outputs were set by
    // the preparation)
    if (threadIdx.x == 0) {
      P.total_latency[k] = 0;
      if (P.makespan) P.makespan[k] = 0;
      if (P.request_steps) P.request_steps[k] = 0;
      if (P.total_evictions) P.total_evictions[k] = 0;
      P.status[k] = st0;
    }
    return;
  }
  using ST = WaveStateWide;
  ST st;
  fresh_state(st, arr_ptr);
  int r;
  do {
    switch (st.next_rows) {
      case 2: r = wave_instance<ALGO, 2, true, true, false, false, ST>(P, k, SCHED_OK, P.retry_status, &st); break;
      case 3: r = wave_instance<ALGO, 3, true, true, false, false, ST>(P, k, SCHED_OK, P.retry_status, &st); break;
      case 5: r = wave_instance<ALGO, 5, true, true, false, false, ST>(P, k, SCHED_OK, P.retry_status, &st); break;
      case 8: r = wave_instance<ALGO, 8, true, true, false, false, ST>(P, k, SCHED_OK, P.retry_status, &st); break;
      case 10: r = wave_instance<ALGO, 10, true, true, false, false, ST>(P, k, SCHED_OK, P.retry_status, &st); break;
      case 12: r = wave_instance<ALGO, 12, true, true, false, false, ST>(P, k, SCHED_OK, P.retry_status, &st); break;
      default: r = wave_instance<ALGO, 16, true, true, false, false, ST>(P, k, SCHED_OK, P.retry_status, &st); break;
    }
  } while (r == kResume);
  finish_instance(P, k, SCHED_OK, r, st.rsteps, st.tot_ev, false);
}

// The narrow ladder: one wave per instance moving along the bodies of 2 to
// 10 rows (the body of the two kernels below; ORDERED_: workgroup g simulates
// instance P.order[g]; CLS_: issue priorities by P.pclass; PRIO_ false: the
// waves keep the default issue priority, for batches in which priorities
// cannot help (a wave per SIMD, or rounds of waves) but would cost scalar
// instructions).  A running set beyond 640 runs ends with P.retry_status.
#define SK_NARROW_LADDER(ORDERED_, CLS_, PRIO_)                                                                                               \
  const int k = (ORDERED_) ? P.order[blockIdx.x] : static_cast<int>(blockIdx.x);                                                       \
  if (P.algo_of && P.algo_of[k] != ALGO) return;                                                                                       \
  const int st0 = P.status[k];                                                                                                         \
  int arr_ptr = 0;                                                                                                                 \
  if (st0 == SCHED_OK) {                                                                                                               \
    /* the bodies all resume from a state, so the bitmaps and staged outputs */                                                        \
    /* are set up here */                                                                                                              \
    extern __shared__ uint64_t lds64[];                                                                                                \
    const int64_t b = P.offsets[k];                                                                                                    \
    const int n = static_cast<int>(P.offsets[k + 1] - b);                                                                              \
    arr_ptr = start_waiting(P, b, n, lds64, lds64 + P.nw_max);                                                                          \
    int32_t* lc = reinterpret_cast<int32_t*>(lds64 + P.nw_max + P.nw1_max + P.cap_v);                                                  \
    if (P.stage_comp)                                                                                                                  \
      for (int i = threadIdx.x; i < n; i += 64) lc[i] = -1;                                                                            \
    __syncthreads();                                                                                                                   \
  }                                                                                                                                    \
  const bool empty = st0 == SCHED_OK && P.offsets[k + 1] == P.offsets[k];                                                              \
  if (st0 != SCHED_OK || empty) {                                                                                                      \
    /* nothing to simulate: zero totals (the per-request outputs were set by */                                                        \
    /* the preparation) */                                                                                                             \
    if (threadIdx.x == 0) {                                                                                                            \
      P.total_latency[k] = 0;                                                                                                          \
      if (P.makespan) P.makespan[k] = 0;                                                                                               \
      if (P.request_steps) P.request_steps[k] = 0;                                                                                     \
      if (P.total_evictions) P.total_evictions[k] = 0;                                                                                 \
      P.status[k] = st0;                                                                                                               \
    }                                                                                                                                  \
    return;                                                                                                                            \
  }                                                                                                                                    \
  WaveState st;                                                                                                                         \
  fresh_state(st, arr_ptr);                                                                                                                  \
  int r;                                                                                                                               \
  do {                                                                                                                                 \
    switch (st.next_rows) {                                                                                                            \
      case 2: r = wave_instance<ALGO, 2, true, true, false, false, WaveState, (CLS_), (PRIO_)>(P, k, SCHED_OK, P.retry_status, &st); break;    \
      case 3: r = wave_instance<ALGO, 3, true, true, false, false, WaveState, (CLS_), (PRIO_)>(P, k, SCHED_OK, P.retry_status, &st); break;    \
      case 5: r = wave_instance<ALGO, 5, true, true, false, false, WaveState, (CLS_), (PRIO_)>(P, k, SCHED_OK, P.retry_status, &st); break;    \
      case 8: r = wave_instance<ALGO, 8, true, true, false, false, WaveState, (CLS_), (PRIO_)>(P, k, SCHED_OK, P.retry_status, &st); break;    \
      default: r = wave_instance<ALGO, 10, true, true, false, false, WaveState, (CLS_), (PRIO_)>(P, k, SCHED_OK, P.retry_status, &st); break;  \
    }                                                                                                                                  \
  } while (r == kResume);                                                                                                              \
  finish_instance(P, k, SCHED_OK, r, st.rsteps, st.tot_ev, false);

// The narrow ladder held to 128 VGPRs so that four waves share a SIMD; each
// (ORDERED, CLS, PRIO) choice is an instance of the kernel of its own, so
// that the other launches compile without it.
template <int ALGO, bool ORDERED = false, bool CLS = false, bool PRIO = true>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_simulate_ladder(Params P) {
  SK_NARROW_LADDER(ORDERED, CLS, PRIO);
}

// The same bodies with 256 VGPRs (fewer spills), for batches in which every
// wave has a SIMD to itself (so without issue priorities).
template <int ALGO>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_simulate_ladder_roomy(Params P) {
  SK_NARROW_LADDER(false, false, false);
}
#undef SK_NARROW_LADDER

// The wide ladder (up to 1024 runs): for batches of few instances, where
// registers matter more than occupancy, and for the instances that outgrow
// the narrow ladder (a retry pass).
template <int ALGO>
__global__ __launch_bounds__(64) void k_simulate_ladder_wide(Params P) {
  wide_ladder_instance<ALGO>(P, blockIdx.x);
}

// The one-wave kernels of a policy, each policy's in a translation unit of its
// own (sched_wave_*.hip): EACH(...) instantiates them there, with `extern`
// before it they are declared to the host code that launches them.
#define SK_WAVE_KERNELS(EACH, ALGO)                                            \
  EACH template __global__ void k_simulate<ALGO, 1, false>(Params);            \
  EACH template __global__ void k_simulate<ALGO, 2, false>(Params);            \
  EACH template __global__ void k_simulate<ALGO, 4, false>(Params);            \
  EACH template __global__ void k_simulate<ALGO, 5, false>(Params);            \
  EACH template __global__ void k_simulate<ALGO, 6, false>(Params);            \
  EACH template __global__ void k_simulate<ALGO, 8, false>(Params);            \
  EACH template __global__ void k_simulate<ALGO, 16, false>(Params);           \
  EACH template __global__ void k_simulate<ALGO, 8, true>(Params);             \
  EACH template __global__ void k_simulate<ALGO, 16, true>(Params);            \
  EACH template __global__ void k_simulate_ladder<ALGO>(Params);               \
  EACH template __global__ void k_simulate_ladder<ALGO, false, false, false>(Params); \
  EACH template __global__ void k_simulate_ladder_roomy<ALGO>(Params);
#define SK_WAVE_KERNELS_AMIN(EACH)                                             \
  SK_WAVE_KERNELS(EACH, SCHED_AMIN)                                            \
  EACH template __global__ void k_simulate<SCHED_AMIN, 16, true, true>(Params); \
  EACH template __global__ void k_simulate_ladder<SCHED_AMIN, true, false, false>(Params); \
  EACH template __global__ void k_simulate_ladder<SCHED_AMIN, false, true>(Params);

}  // namespace sk
