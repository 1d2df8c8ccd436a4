// sim_tiny.hpp -- many tiny instances: one lane simulates one instance (device
// code of k_tiny).
//
// What bounds it: with at most eight requests an instance has a few dozen events,
// so a wave per instance spends its time on the preparation and its launch
// rather than on lanes that work.  Here one launch does all of it: a lane reads its
// instance, validates it, holds every request in registers and steps from event
// to event, with the planned memory summed anew for every test (64 terms, no state
// to keep).  The lanes of a wave go through their own events together, so a wave
// lasts as long as its longest instance (about 0.12 ms at six requests), which
// pays once the device would go through several rounds of one-instance waves.
// 262144 instances of 6 requests, A_min: 0.21 ms (a wave per instance: 1.09 ms);
// 16384 of them: 0.12 ms (0.10 ms).
#pragma once

#include "sim_device.hpp"

namespace sk {

// most requests of an instance that a lane holds
constexpr int kTinyRequests = 8;

// (held to 128 registers so that four waves share a SIMD)
template <int ALGO>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_tiny(Params P) {
  constexpr int NM = kTinyRequests;
  const int k = blockIdx.x * 64 + static_cast<int>(threadIdx.x);
  if (k >= P.K) return;
  const int64_t b = P.offsets[k];
  const int64_t e = P.offsets[k + 1];
  const bool range = b >= 0 && e >= b && e <= P.N && e - b <= P.max_requests;
  const int n = range ? static_cast<int>(e - b) : 0;
  const int32_t M = P.M;
  constexpr bool kReadL = ALGO == SCHED_AMIN || ALGO == SCHED_AELL || ALGO == SCHED_ADAPTIVE;
  constexpr bool kReadU = ALGO == SCHED_AMAX || ALGO == SCHED_AELL || ALGO == SCHED_ADAPTIVE;
  constexpr bool kReadP = ALGO == SCHED_ARANDOM;
  constexpr int32_t kNoStep = 0x7FFFFFFF;

  // ---- the requests, and the checks of validate_instance
  int32_t a[NM], s[NM], o[NM], lo[NM], up[NM], tk[NM], pr[NM];
  bool arr_bad = false, int_bad = false, big_bad = false, unsup = false;
  bool bad_l = false, unsup_l = false, bad_u = false, big_u = false, unsup_u = false;
  int64_t sum_o = 0, sum_l = 0, sum_u = 0;
  int32_t max_a = 0, prev = 0;
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    a[i] = 0; s[i] = 0; o[i] = 1; lo[i] = 1; up[i] = 1; tk[i] = 0; pr[i] = 0;
    if (i < n) {
      if (P.arrival) a[i] = P.arrival[b + i];
      s[i] = P.prompt[b + i];
      o[i] = P.output[b + i];
      if (kReadL) lo[i] = P.lower[b + i];
      if (kReadU) up[i] = P.upper[b + i];
      if (kReadP) pr[i] = P.priority[b + i];
      if (P.tie_key) tk[i] = P.tie_key[b + i];
      arr_bad = arr_bad || a[i] < 0 || (i > 0 && a[i] < prev);
      prev = a[i];
      int_bad = int_bad || o[i] < 1 || s[i] < 0;
      bad_l = bad_l || lo[i] < 1 || lo[i] > o[i];
      bad_u = bad_u || up[i] < o[i];
      big_bad = big_bad || static_cast<int64_t>(s[i]) + o[i] > M;
      big_u = big_u || static_cast<int64_t>(s[i]) + up[i] > M;
      unsup = unsup || o[i] >= kEstLimit || s[i] >= kPromptLimit || pr[i] < 0 || pr[i] >= kEstLimit;
      unsup_l = unsup_l || lo[i] >= kEstLimit;
      unsup_u = unsup_u || up[i] >= kEstLimit;
      max_a = a[i] > max_a ? a[i] : max_a;
      sum_o += static_cast<int64_t>(o[i]) + 1;
      sum_l += lo[i];
      sum_u += up[i];
    }
  }
  int algo = ALGO;
  if (ALGO == SCHED_ADAPTIVE) {
    const int64_t d = 3 * sum_u - 2 * sum_l;
    algo = SCHED_AMIN;
    if (n > 0 && d > 0) {
      const unsigned __int128 dd = static_cast<unsigned __int128>(d) * static_cast<unsigned __int128>(d);
      const unsigned __int128 uu = static_cast<unsigned __int128>(sum_u) * static_cast<unsigned __int128>(sum_u);
      if (dd > 5 * uu) algo = SCHED_AELL;
    }
  }
  const bool amin = algo == SCHED_AMIN, aell = algo == SCHED_AELL;
  const bool use_l = amin || aell, use_u = algo == SCHED_AMAX || aell;
  int status = !range                                                            ? SCHED_E_INVAL
               : arr_bad                                                         ? SCHED_E_ARRIVAL
               : int_bad || (use_l && bad_l) || (use_u && bad_u)                 ? SCHED_E_INTERVAL
               : big_bad || (use_u && big_u)                                     ? SCHED_E_TOO_BIG
               : unsup || (use_l && unsup_l) || (use_u && unsup_u) ? SCHED_E_UNSUPPORTED
                                                                                 : SCHED_OK;
  int64_t cap64 = P.step_cap > 0 ? P.step_cap : 4 * (static_cast<int64_t>(max_a) + sum_o) + 64;
  if (cap64 > kCapLimit) cap64 = kCapLimit;
  const int32_t cap = static_cast<int32_t>(cap64);

  // ---- state: planned length, place in the order of the waiting requests (and of
  // the cancellations), x = s - start, planned end and completion of a run, counts
  int32_t est[NM], x[NM], end[NM], done[NM], evs[NM];
  uint32_t ord[NM], rank[NM];
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    // the tie rank: by (tie key, index), A_l's by (arrival, tie key, index)
    uint32_t r = 0;
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      const bool tie_less = tk[j] < tk[i] || (tk[j] == tk[i] && j < i);
      const bool less = aell ? a[j] < a[i] || (a[j] == a[i] && tie_less) : tie_less;
      r += (j != i && j < n && less) ? 1u : 0u;
    }
    rank[i] = r;
    const int32_t key = algo == SCHED_AMAX ? up[i] : algo == SCHED_ARANDOM ? pr[i] : use_l ? lo[i] : o[i];
    est[i] = algo == SCHED_ARANDOM ? o[i] : key;
    ord[i] = aell ? r : (static_cast<uint32_t>(key) << 5) | r;
    x[i] = 0; end[i] = 0; done[i] = -1; evs[i] = 0;
  }
  // memory at step c of N runs whose s - start sum to x (the product may wrap round)
  auto at = [](int32_t sx, int32_t nr, int32_t c) {
    return static_cast<int32_t>(static_cast<uint32_t>(sx) + static_cast<uint32_t>(nr) * static_cast<uint32_t>(c));
  };
  const uint32_t all = n > 0 ? (1u << n) - 1u : 0u;
  uint32_t coming = status == SCHED_OK ? all : 0u;   // not arrived yet
  uint32_t waits = 0, runs = 0, gated = 0;           // gated: cancelled at this step
  uint32_t promoted = 1u << 20;                      // the next promoted request's place
  int32_t t = 0;
  int64_t rsteps = 0, tot_ev = 0;
  while (coming | waits | runs | gated) {
    if (t > cap) {
      status = SCHED_E_STEP_CAP;
      break;
    }
    // arrivals, last step's cancellations, completions
    waits |= gated;
    gated = 0;
    int32_t next = kNoStep;       // the next event
    int32_t DT = 0;
    int32_t N = 0, X = 0;         // runs, and the sum of their s - start
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      const uint32_t bit = 1u << i;
      if (coming & bit) {
        if (a[i] <= t) {
          coming ^= bit;
          waits |= bit;
        } else {
          next = a[i] < next ? a[i] : next;
        }
      }
      if (runs & bit) {
        if (done[i] == t) {
          runs ^= bit;
          DT += x[i] + t;
        } else {
          N += 1;
          X = static_cast<int32_t>(static_cast<uint32_t>(X) + static_cast<uint32_t>(x[i]));
        }
      }
    }
    if (!(coming | waits | runs)) break;
    if (ALGO == SCHED_AELL || ALGO == SCHED_ADAPTIVE) {
      // promotions: runs present at their planned end, in tie-rank order
      for (;;) {
        uint32_t bi = NM, br = ~0u;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          const bool due = aell && ((runs >> i) & 1u) && end[i] == t && rank[i] < br;
          br = due ? rank[i] : br;
          bi = due ? i : bi;
        }
        if (bi == NM) break;
#pragma unroll
        for (int i = 0; i < NM; ++i)
          if (static_cast<uint32_t>(i) == bi) {
            runs ^= 1u << i;
            waits |= 1u << i;
            N -= 1;
            X = static_cast<int32_t>(static_cast<uint32_t>(X) - static_cast<uint32_t>(x[i]));
            est[i] = up[i];
            ord[i] = promoted;
            done[i] = -1;
            evs[i] += 1;
          }
        ++promoted;
        ++tot_ev;
      }
    }
    if (ALGO == SCHED_AMIN || ALGO == SCHED_ADAPTIVE) {
      // cancel in ascending (planned length, rank) while the memory at t+1 is above M
      while (amin && at(X, N, t + 1) > M) {
        uint32_t bi = 0, bo = ~0u;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          const bool less = ((runs >> i) & 1u) && ord[i] < bo;
          bo = less ? ord[i] : bo;
          bi = less ? i : bi;
        }
#pragma unroll
        for (int i = 0; i < NM; ++i)
          if (static_cast<uint32_t>(i) == bi) {
            runs ^= 1u << i;
            gated |= 1u << i;
            N -= 1;
            X = static_cast<int32_t>(static_cast<uint32_t>(X) - static_cast<uint32_t>(x[i]));
            const int32_t gen = t - (end[i] - est[i]);
            est[i] = gen > est[i] ? gen : est[i];
            ord[i] = (static_cast<uint32_t>(est[i]) << 5) | rank[i];
            done[i] = -1;
            evs[i] += 1;
          }
        ++tot_ev;
      }
    }
    // admissions; wait_until: the step before which the head cannot start (kNoStep:
    // not before another event)
    int32_t wait_until = kNoStep;
    while (waits) {
      uint32_t bi = 0, bo = ~0u;
      int32_t cs = 0, co = 0, ce = 0;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        const bool less = ((waits >> i) & 1u) && ord[i] < bo;
        bo = less ? ord[i] : bo;
        bi = less ? i : bi;
        cs = less ? s[i] : cs;
        co = less ? o[i] : co;
        ce = less ? est[i] : ce;
      }
      if (at(X, N, t + 1) + cs + 1 > M) break;
      if (DT > 0 && DT + at(X, N, t) + cs > M) {
        wait_until = t + 1;
        break;
      }
      // planned ends c in (t+1, E] gain cs + c - t, and E itself
      const int32_t E = t + ce;
      int32_t fix = 0, fe = cs + ce, emin = kNoStep;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        const bool run = (runs >> i) & 1u;
        const int32_t c = end[i];
        if (run && c >= E) {
          fe += x[i] + E;
          emin = c < emin ? c : emin;
        }
        if (run && c > t + 1 && c <= E) {
          int32_t f = cs + c - t;
#pragma unroll
          for (int j = 0; j < NM; ++j) f += ((runs >> j) & 1u) && end[j] >= c ? x[j] + c : 0;
          const int32_t over = f - M, left = c - 1 - t;
          const int32_t m = over < left ? over : left;
          fix = over > 0 && m > fix ? m : fix;
        }
      }
      if (fix > 0) {
        wait_until = t + fix;
        break;
      }
      if (ce > 1 && fe > M) {
        wait_until = emin - ce + 1;
        break;
      }
#pragma unroll
      for (int i = 0; i < NM; ++i)
        if (static_cast<uint32_t>(i) == bi) {
          x[i] = cs - t;
          end[i] = E;
          done[i] = t + co;
        }
      waits ^= 1u << bi;
      runs |= 1u << bi;
      N += 1;
      X = static_cast<int32_t>(static_cast<uint32_t>(X) + static_cast<uint32_t>(cs - t));
    }
    rsteps += N;
    // the next step at which something can happen
    int32_t tn = t + 1;
    if (!gated) {
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        if ((runs >> i) & 1u) {
          next = done[i] < next ? done[i] : next;
          if (aell) next = end[i] < next ? end[i] : next;
        }
      }
      next = wait_until < next ? wait_until : next;
      next = cap + 1 < next ? cap + 1 : next;
      if (amin && N > 0) {
        const int32_t Pm = at(X, N, t + 1);   // <= M here
        if (static_cast<int64_t>(Pm) + static_cast<int64_t>(N) * (next - 1 - t) > M) {
          const int32_t tev = t + (M - Pm) / N + 1;
          next = tev < next ? tev : next;
        }
      }
      if (next > tn) {
        rsteps += static_cast<int64_t>(N) * (next - tn);
        tn = next;
      }
    }
    t = tn;
  }
  // ---- outputs: a run that has not ended has no completion step
  int64_t tel = 0;
  int32_t mk = 0;
  const bool keep = status == SCHED_OK || status == SCHED_E_STEP_CAP;
  const uint32_t left = coming | waits | runs | gated;
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    if (i < n) {
      const int32_t c = keep && !((left >> i) & 1u) ? done[i] : -1;
      P.completion[b + i] = c;
      if (P.evictions) P.evictions[b + i] = keep ? evs[i] : 0;
      if (c >= 0) {
        tel += c - a[i];
        mk = c > mk ? c : mk;
      }
    }
  }
  P.total_latency[k] = tel;
  P.status[k] = status;
  if (P.makespan) P.makespan[k] = mk;
  if (P.request_steps) P.request_steps[k] = keep ? rsteps : 0;
  if (P.total_evictions) P.total_evictions[k] = keep ? tot_ev : 0;
  if (P.algo_used) P.algo_used[k] = algo;
}

}  // namespace sk
