// sched_kernels.hip -- the C ABI of the scheduler simulator (host side), the
// preparation and launch-order kernels and, unless SK_SEPARATE_KERNELS leaves
// them to sched_wave_*.hip (built concurrently), the one-wave kernels.  The wide
// row ladder (sched_wide.hip) and the workgroup kernels (sched_group*.hip) are
// translation units of their own.  The device code is in sim_wave.hpp and
// sim_device.hpp.
#include "prepare.hpp"
#include "sim_tiny.hpp"
#include "sim_wave.hpp"

namespace sk {
#ifdef SK_SEPARATE_KERNELS
// defined in sched_wave_*.hip (else here)
SK_WAVE_KERNELS(extern, SCHED_AMAX)
SK_WAVE_KERNELS_AMIN(extern)
SK_WAVE_KERNELS(extern, SCHED_HSF)
SK_WAVE_KERNELS(extern, SCHED_AELL)
SK_WAVE_KERNELS(extern, SCHED_ARANDOM)
#endif
// defined in sched_wide.hip
extern template __global__ void k_simulate_ladder_wide<SCHED_AMAX>(Params);
extern template __global__ void k_simulate_ladder_wide<SCHED_AMIN>(Params);
extern template __global__ void k_simulate_ladder_wide<SCHED_HSF>(Params);
extern template __global__ void k_simulate_ladder_wide<SCHED_AELL>(Params);
extern template __global__ void k_simulate_ladder_wide<SCHED_ARANDOM>(Params);
// defined in sched_group.hip
SK_GROUP_KERNELS(extern)
SK_GROUP_KERNELS_AMIN(extern)

// One wave an instance that sleeps until all of them have started (about 2 us).  A
// CU gives a new wave the SIMD that follows the last one's, as long as waves end in the
// order in which they came: after a kernel whose workgroups have several waves, or come
// one after the other for lack of LDS, the CU's next four waves may share SIMDs (3 to 10
// in 100 of 1024 waves on 256 CUs did, none after this kernel).  A simulation lasts as
// long as its slowest instance, and a wave that shares its SIMD is slower: 1024 x 10000
// A_l took 26.9 ms instead of 22.9, A_min 27.0 instead of 24.1.  Where it is
// launched: prepare_launch.
__global__ __launch_bounds__(64) void k_spread() { __builtin_amdgcn_s_sleep(64); }

// Issue-priority classes (A_min with upper bounds, from k_prepare): kept only
// where they differ between the instances of the batch; a batch whose
// instances share one class keeps the priority by unfinished work alone.
__global__ __launch_bounds__(256) void k_prio_classes(Params P) {
  __shared__ int lo_s, hi_s;
  if (threadIdx.x == 0) {
    lo_s = 3;
    hi_s = -1;
  }
  __syncthreads();
  int lo = 3, hi = -1;
  for (int k = threadIdx.x; k < P.K; k += 256) {
    const int c = P.pclass[k];
    if (c < 3) {
      lo = c < lo ? c : lo;
      hi = c > hi ? c : hi;
    }
  }
  atomicMin(&lo_s, lo);
  atomicMax(&hi_s, hi);
  __syncthreads();
  if (lo_s >= hi_s)
    for (int k = threadIdx.x; k < P.K; k += 256) P.pclass[k] = -1;
}

// The instances that a retry pass takes, in no particular order (algo: the policy
// of the pass, in adaptive runs).  All are counted, those that the list has room for
// are listed.
__global__ __launch_bounds__(256) void k_retry_list(Params P, RetryList R, int algo) {
  const int k = blockIdx.x * 256 + static_cast<int>(threadIdx.x);
  const int lane = static_cast<int>(threadIdx.x & 63u);
  const bool take = k < P.K && !(P.algo_of && P.algo_of[k] != algo) && retry_takes(P, P.status[k]);
  const uint64_t m = __builtin_amdgcn_ballot_w64(take);
  if (m == 0) return;
  int base = 0;
  if (lane == 0) base = atomicAdd(&R.count[0], __builtin_popcountll(m));
  base = __builtin_amdgcn_readfirstlane(base);
  const int at = base + __builtin_popcountll(m & ((1ull << lane) - 1ull));
  if (take && at < R.room) R.list[at] = k;
}

// Launch order (A_min batches served in several rounds of waves): the
// instances by decreasing key, so that the longest expected simulations are
// not the last ones to start.  The order within a bucket is whatever the
// atomics give; outputs do not depend on the order.
__global__ __launch_bounds__(64) void k_order_clear(Params P) {
  P.obucket[threadIdx.x] = 0;
}
__global__ __launch_bounds__(64) void k_order_scan(Params P) {
  // bucket b starts after every bucket above it
  if (threadIdx.x == 0) {
    int32_t run = 0;
    for (int b = kOrderBuckets - 1; b >= 0; --b) {
      const int32_t c = P.obucket[b];
      P.obucket[b] = run;
      run += c;
    }
  }
}
__global__ __launch_bounds__(256) void k_order_scatter(Params P) {
  // one atomic per distinct key of a wave (neighbouring instances mostly
  // share their key), the lanes of a key placed in lane order
  const int k = blockIdx.x * 256 + static_cast<int>(threadIdx.x);
  const int lane = static_cast<int>(threadIdx.x & 63u);
  const bool act = k < P.K;
  const int key = act ? P.okey[k] : -1;
  uint64_t left = __builtin_amdgcn_ballot_w64(act);
  while (left) {
    const int lead = __builtin_ctzll(left);
    const int lkey = __builtin_amdgcn_readlane(key, lead);
    const uint64_t same = __builtin_amdgcn_ballot_w64(act && key == lkey) & left;
    int base = 0;
    if (lane == lead) base = atomicAdd(&P.obucket[lkey], __builtin_popcountll(same));
    base = __builtin_amdgcn_readlane(base, lead);
    if ((same >> lane) & 1ull) {
      const int below = __builtin_popcountll(same & ((1ull << lane) - 1ull));
      P.order[base + below] = k;
    }
    left &= ~same;
  }
}
}  // namespace sk

// ---------------------------------------------------------------------------
// The workspace of sched_simulate_noalloc: a fixed array in device memory
// (each device that runs the library holds its own copy until the process
// ends).  Host code never passes `scratch` itself to a kernel or a copy (in
// host code the name is a host-side stand-in): it uses the device address
// that hipGetSymbolAddress returns, taken once per device.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = size_t(96) << 20;
// (beyond a call's workspace, the retry passes' counts)
constexpr size_t kRetryBytes = 4 * sk::kRetryCounts;
static __device__ __align__(256) unsigned char scratch[kScratchBytes + kRetryBytes];

// ---------------------------------------------------------------------------
// host side: the C ABI
// ---------------------------------------------------------------------------
namespace {

// Device address of `scratch` on device `dev` (the current device), looked up
// on the first call on that device and kept.
hipError_t scratch_address(int dev, void** out) {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static void* addr[kMaxDev] = {};
  if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

// One launch of the simulation kernel over the batch.
struct Tier {
  int rows;         // register rows (fixed-row kernels; per wave in a workgroup)
  bool grow;        // a row ladder: k_simulate_ladder, or k_simulate_ladder_wide with wide
  bool wide;
  bool retry;       // a retry pass: runs the instances an earlier pass handed over (run_mask)
  bool vglobal;     // cancelled set in global memory (16 rows)
  int cap_v;        // LDS slots of the cancelled set (LDS passes)
  int run_mask;     // retry: bit 0 takes kRetryRows, bit 1 kRetryV
  int rows_status;  // status for an outgrown running set
  int v_status;     // status for an outgrown cancelled set
  int stage;        // completion steps staged in LDS (1) or not (0)
  int gw;           // > 1: a workgroup of gw waves per instance (k_simulate_group)
  int grid;         // workgroups of the launch (0: one per instance)
  int roomy;        // the narrow ladder with 256 VGPRs (k_simulate_ladder_roomy)
  int list;         // a retry pass over a list of the instances that it takes (k_retry_list)
};

// The workgroup kernels that exist (sched_group*.hip), else NULL.  list: over a list of
// the instances (retry passes).
template <int ALGO, int W, bool VGLOBAL>
const void* group_retry_kernel(bool list) {
  return list ? reinterpret_cast<const void*>(&sk::k_simulate_group_listed<ALGO, W, VGLOBAL>)
              : reinterpret_cast<const void*>(&sk::k_simulate_group<ALGO, W, 16, VGLOBAL>);
}

template <int ALGO, bool VGLOBAL>
const void* group_first_kernel(int w) {
  return w == 2 ? reinterpret_cast<const void*>(&sk::k_simulate_group<ALGO, 2, 8, VGLOBAL>)
                : reinterpret_cast<const void*>(&sk::k_simulate_group<ALGO, 4, 4, VGLOBAL>);
}

template <int ALGO>
const void* group_kernel(int w, int rows, bool vglobal, bool list) {
  const bool first = (w == 2 && rows == 8) || (w == 4 && rows == 4);
  if (!first && (rows != 16 || (w != 4 && w != 8))) return nullptr;
  if (first && list) return nullptr;
  if constexpr (ALGO == SCHED_AMIN) {
    if (first) return vglobal ? group_first_kernel<ALGO, true>(w) : group_first_kernel<ALGO, false>(w);
    if (w == 8) return vglobal ? group_retry_kernel<ALGO, 8, true>(list) : nullptr;
    return vglobal ? group_retry_kernel<ALGO, 4, true>(list) : group_retry_kernel<ALGO, 4, false>(list);
  } else {
    if (vglobal) return nullptr;
    if constexpr (ALGO == SCHED_AMAX || ALGO == SCHED_HSF)
      if (first) return group_first_kernel<ALGO, false>(w);
    if (first) return nullptr;
    return w == 8 ? group_retry_kernel<ALGO, 8, false>(list) : group_retry_kernel<ALGO, 4, false>(list);
  }
}

template <int ALGO>
const void* sim_kernel(const Tier& tr, bool ordered, bool classes, bool rounds) {
  if (tr.gw > 1) return group_kernel<ALGO>(tr.gw, tr.rows, tr.vglobal, tr.list != 0);
  if constexpr (ALGO == SCHED_AMIN) {
    if (tr.grow && !tr.wide && ordered)
      return reinterpret_cast<const void*>(&sk::k_simulate_ladder<ALGO, true, false, false>);
    if (tr.grow && !tr.wide && classes)
      return reinterpret_cast<const void*>(&sk::k_simulate_ladder<ALGO, false, true>);
  }
  if (tr.grow && !tr.wide && tr.roomy) return reinterpret_cast<const void*>(&sk::k_simulate_ladder_roomy<ALGO>);
  if (tr.grow && !tr.wide && rounds)
    return reinterpret_cast<const void*>(&sk::k_simulate_ladder<ALGO, false, false, false>);
  if (tr.grow)
    return tr.wide ? reinterpret_cast<const void*>(&sk::k_simulate_ladder_wide<ALGO>)
                   : reinterpret_cast<const void*>(&sk::k_simulate_ladder<ALGO>);
  if constexpr (ALGO == SCHED_AMIN)
    if (tr.vglobal) return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 16, true, true>);
  if (tr.retry)
    return tr.rows <= 8    ? reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 8, true>)
                           : reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 16, true>);
  switch (tr.rows) {
    case 1: return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 1, false>);
    case 2: return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 2, false>);
    case 4: return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 4, false>);
    case 5: return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 5, false>);
    case 6: return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 6, false>);
    case 8: return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 8, false>);
    default: return reinterpret_cast<const void*>(&sk::k_simulate<ALGO, 16, false>);
  }
}

// The preparation's kernel, its waves an instance and its dynamic LDS.
struct PrepareLaunch {
  const void* kernel;
  int waves;
  size_t lds;
  bool spread;  // k_spread has to follow
};

template <int W, bool LDS>
const void* prepare_kernel(int algo) {
  switch (algo) {
    case SCHED_AMAX: return reinterpret_cast<const void*>(sk::k_prepare<SCHED_AMAX, W, LDS>);
    case SCHED_AMIN: return reinterpret_cast<const void*>(sk::k_prepare<SCHED_AMIN, W, LDS>);
    case SCHED_HSF: return reinterpret_cast<const void*>(sk::k_prepare<SCHED_HSF, W, LDS>);
    case SCHED_AELL: return reinterpret_cast<const void*>(sk::k_prepare<SCHED_AELL, W, LDS>);
    case SCHED_ARANDOM: return reinterpret_cast<const void*>(sk::k_prepare<SCHED_ARANDOM, W, LDS>);
    default: return reinterpret_cast<const void*>(sk::k_prepare<SCHED_ADAPTIVE, W, LDS>);
  }
}

// One wave an instance where it is one or a few chunks of 64 requests (with more
// waves, most of them would wait at barriers), else four while an instance's buffers let
// a CU hold several workgroups of them, else sixteen.  Measured, with 1 / 4 / 16
// waves an instance: 65536 x 2000 2.32 / 1.45 / 3.84 ms, 1024 x 10000 0.79 / 0.43 /
// 0.27 ms, 3000 x 1500 with tie keys 173 / 87 / 325 us, 4096 x 1000 58 / 50 / 192 us.
// k_spread takes 2 to 5 us of the call.  With it, against without, on 256 CUs: 1500 to 3000
// requests 0.85 to 0.92 of the time at 1024 and 2048 instances, 0.89 to 0.96 at 3072, 0.98 to 1.01
// at the counts between (a CU's last SIMDs then hold one wave fewer than the others
// anyway) but 0.91 for 2816 of A_l; 300 to 1000 requests 1.00 to 1.03 up to 2560, 0.89 to 0.97 at
// 3072, 0.93 to 1.03 at 2816.  Above 12 a CU some SIMD has four waves in any order: 1.00 to 1.02.
PrepareLaunch prepare_launch(int algo, int64_t nmax, int64_t K, int n_cu, bool tie, int lds_max) {
  // A_l sorts nothing but tie keys
  const size_t lds = (tie ? 12 : algo == SCHED_AELL ? 4 : 8) * static_cast<size_t>(std::max<int64_t>(nmax, 1));
  if (nmax <= 64 || (nmax <= 256 && K > 2 * int64_t(n_cu))) return {prepare_kernel<1, true>(algo), 1, lds, false};
  const bool spread = K <= 12 * int64_t(n_cu) && K > (nmax > 1024 ? 2 : 8) * int64_t(n_cu);
  if (nmax <= 4096) return {prepare_kernel<4, true>(algo), 4, lds, spread};
  if (lds + sizeof(sk::PrepareShared<16>) <= static_cast<size_t>(lds_max))
    return {prepare_kernel<16, true>(algo), 16, lds, spread};
  return {prepare_kernel<16, false>(algo), 16, 0, spread};
}

// ordered: A_min's narrow ladder takes the instances in the order P.order;
// classes: it sets issue priorities by P.pclass; rounds: the batch is served
// in rounds of waves (the narrow ladder without issue priorities)
const void* sim_kernel_any(int algo, const Tier& tr, bool ordered = false, bool classes = false,
                           bool rounds = false) {
  switch (algo) {
    case SCHED_AMAX: return sim_kernel<SCHED_AMAX>(tr, false, false, rounds);
    case SCHED_AMIN: return sim_kernel<SCHED_AMIN>(tr, ordered, classes, rounds);
    case SCHED_HSF: return sim_kernel<SCHED_HSF>(tr, false, false, rounds);
    case SCHED_ARANDOM: return sim_kernel<SCHED_ARANDOM>(tr, false, false, rounds);
    default: return sim_kernel<SCHED_AELL>(tr, false, false, rounds);
  }
}

// register rows that hold `want` runs
int rows_for(int64_t want) {
  const int64_t r = (want + 63) / 64;
  return r <= 1 ? 1 : r <= 2 ? 2 : r <= 4 ? 4 : r <= 5 ? 5 : r <= 6 ? 6 : r <= 8 ? 8 : 16;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// The LDS of a launch: the bitmaps' words and the most a workgroup holds.
struct Room {
  size_t lds_max;
  int nw, nw1;
};

// LDS bytes of a workgroup launch (W waves, `rows` rows each) whose waves
// each hold cap_v cancelled-set slots (0: a global set), staging aside.
size_t group_lds(int algo, int w, int rows, const Room& rm, int cap_v) {
  return 8 * (static_cast<size_t>(sk::group_pre_words(algo, w, rows)) +
              static_cast<size_t>(w) * (static_cast<size_t>(rm.nw) + rm.nw1 + cap_v));
}

// Cancelled-set slots per wave that the LDS of such a launch leaves room for
// (-1: not even the bitmaps fit).
int64_t group_cap_fit(int algo, int w, int rows, const Room& rm) {
  const size_t base = group_lds(algo, w, rows, rm, 0);
  return base > rm.lds_max ? -1 : static_cast<int64_t>((rm.lds_max - base) / (8 * static_cast<size_t>(w)));
}

// The launches that simulate a batch under one policy.  The first holds an
// instance's running set in register rows whose number follows it (the row
// ladder: 2, 3, 5, 8, 10 rows, four waves a SIMD); an instance that needs more
// than 640 runs is simulated again from step 0 by the wide ladder (12 and 16
// more rows, 1024 runs, fewer waves a SIMD), which is also the first launch of a
// batch of few instances that may need it; one that needs more than 1024 runs,
// by a workgroup of 4 waves with 16 rows each (4096 runs), then of 8 waves
// (8192).  With workgroup_waves = W (2 or 4), the first launch is a workgroup
// of W waves with 1024 / (64 W) rows each instead.  The cancelled set (A_min)
// first gets cap0 LDS slots (a size chosen for occupancy); an instance that
// outgrows them is simulated again with as many slots as a workgroup's LDS
// holds, and one that outgrows those again with a global-memory set of n
// slots (per wave), which always suffices (at most n requests wait
// cancelled).  So whether an instance completes never depends on the other
// instances of the batch or on these sizes: only running sets above 8192 runs
// (4096 where eight waves' bitmaps do not fit the LDS), or above a caller's
// forced running capacity, are refused.
int build_tiers(int algo, int64_t nmax, int64_t K, int forced_rows, int cap0, int cap_fit, int ww, const Room& rm,
                bool simd_each, Tier* out) {
  // (A_l's queue lives in global memory and never overflows)
  const bool has_v = algo == SCHED_AMIN;
  const int64_t need_v = has_v ? std::max<int64_t>(nmax, 1) : 0;
  const int cap1 = has_v ? static_cast<int>(std::min<int64_t>(need_v, cap_fit)) : 0;
  const bool v_retry = has_v && cap0 < need_v && cap1 > cap0;  // a larger LDS set may help
  const bool v_lds_short = has_v && cap1 < need_v;              // even the largest LDS set may not
  int m = 0;
  // a workgroup launch: with an LDS cancelled set when `want` slots per wave
  // fit (and a global-set retry if that may be short), else a global set
  auto group = [&](int w, int rows, int mask) {
    if (!has_v) {
      out[m++] = Tier{rows, false, false, mask != 0, false, 0, mask, 0, 0, 0, w, 0};
      return;
    }
    const int64_t want = std::min<int64_t>(need_v, 16384);
    const int64_t fit = std::min<int64_t>(group_cap_fit(algo, w, rows, rm), cap_fit);
    const bool lds = fit >= want && group_kernel<SCHED_AMIN>(w, rows, false, false) != nullptr;
    if (lds) out[m++] = Tier{rows, false, false, mask != 0, false, static_cast<int>(want), mask, 0, 0, 0, w, 0};
    if (!lds || want < need_v) out[m++] = Tier{rows, false, false, true, true, 0, lds ? 2 : (mask ? mask : 0), 0, 0, 0, w, 0};
  };
  if (ww > 1) {
    group(ww, 1024 / (64 * ww), 0);
  } else if (forced_rows > 0) {
    out[m++] = Tier{forced_rows, false, false, false, false, cap0, 0, 0, 0, 0, 0, 0};
    if (v_retry) out[m++] = Tier{16, false, false, true, false, cap1, 2, 0, 0, 0, 0, 0};
    if (v_lds_short) out[m++] = Tier{16, false, false, true, true, 0, 2, 0, 0, 0, 0, 0};
  } else if (nmax <= 128) {
    out[m++] = Tier{rows_for(std::max<int64_t>(nmax, 1)), false, false, false, false, cap0, 0, 0, 0, 0, 0, 0};
    if (v_retry) out[m++] = Tier{8, false, false, true, false, cap1, 2, 0, 0, 0, 0, 0};
    if (v_lds_short) out[m++] = Tier{16, false, false, true, true, 0, 2, 0, 0, 0, 0, 0};
  } else {
    // few instances of many requests start on the wide ladder (they would
    // likely outgrow the narrow one, and the retry would simulate them again);
    // where every wave has a SIMD to itself (simd_each) the narrow bodies get
    // 256 VGPRs, which costs no occupancy there and spills less
    const bool wide0 = nmax > 4096 && K <= 256;
    out[m++] = Tier{0, true, wide0, false, false, cap0, 0, 0, 0, 0, 0, 0, !wide0 && simd_each ? 1 : 0};
    const int mask = (!wide0 && nmax > 640 ? 1 : 0) | (v_retry ? 2 : 0);
    if (mask) out[m++] = Tier{0, true, true, true, false, cap1, mask, 0, 0, 0, 0, 0};
    if (v_lds_short) out[m++] = Tier{16, false, false, true, true, 0, 2, 0, 0, 0, 0, 0};
  }
  // beyond 1024 runs: workgroups (a forced capacity holds instead)
  if (forced_rows == 0 && nmax > 1024) {
    group(4, 16, 1);
    // eight waves when their bitmaps (and lists) fit the LDS
    if (group_cap_fit(algo, 8, 16, rm) >= 0) {
      if (has_v)
        out[m++] = Tier{16, false, false, true, true, 0, 1, 0, 0, 0, 8, 0};
      else
        out[m++] = Tier{16, false, false, true, false, 0, 1, 0, 0, 0, 8, 0};
    }
  }
  // what a pass writes for an instance it cannot hold: a later pass that takes
  // it, or the final refusal
  for (int p = 0; p < m; ++p) {
    bool later_rows = false, later_v = false;
    for (int q = p + 1; q < m; ++q) {
      later_rows = later_rows || (out[q].run_mask & 1);
      later_v = later_v || (out[q].run_mask & 2);
    }
    out[p].rows_status = later_rows ? sk::kRetryRows : SCHED_E_UNSUPPORTED;
    out[p].v_status = later_v ? sk::kRetryV : SCHED_E_UNSUPPORTED;
  }
  return m;
}

// A second stream per device (default priority, created on first use and kept
// for the life of the process): the adaptive policy runs its A_l launches on
// it while the A_min launches run on the caller's stream.  The two touch
// disjoint instances.
hipError_t side_stream(int dev, hipStream_t* out) {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static hipStream_t streams[kMaxDev] = {};
  if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!streams[dev]) {
    const hipError_t e = hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking);
    if (e != hipSuccess) {
      streams[dev] = nullptr;
      return e;
    }
  }
  *out = streams[dev];
  return hipSuccess;
}

// Argument checks shared by the entry points (no HIP call).
int check_args(const sched_instances_t* in, int32_t algo, int64_t M) {
  if (!in) return SCHED_E_INVAL;
  if (algo < SCHED_AMAX || algo > SCHED_ARANDOM) return SCHED_E_INVAL;
  if (M <= 0 || M >= (int64_t(1) << 30)) return SCHED_E_INVAL;
  if (in->num_instances < 0 || in->max_requests < 0 || in->total_requests < 0) return SCHED_E_INVAL;
  if (in->num_instances == 0) return SCHED_OK;
  if (!in->offsets) return SCHED_E_INVAL;
  const bool need_l = algo == SCHED_AMIN || algo == SCHED_AELL || algo == SCHED_ADAPTIVE;
  const bool need_u = algo == SCHED_AMAX || algo == SCHED_AELL || algo == SCHED_ADAPTIVE;
  if (in->total_requests > 0 && (!in->prompt || !in->output)) return SCHED_E_INVAL;
  if (in->total_requests > 0 && need_l && !in->lower) return SCHED_E_INVAL;
  if (in->total_requests > 0 && need_u && !in->upper) return SCHED_E_INVAL;
  if (in->total_requests > 0 && algo == SCHED_ARANDOM && !in->priority) return SCHED_E_INVAL;
  if (in->max_requests >= (1 << sk::kIdxBits)) return SCHED_E_UNSUPPORTED;
  return SCHED_OK;
}

sk::Params base_params(const sched_instances_t* in, int64_t M) {
  sk::Params P{};
  P.K = in->num_instances;
  P.max_requests = in->max_requests;
  P.N = in->total_requests;
  P.offsets = in->offsets;
  P.arrival = in->arrival;
  P.prompt = in->prompt;
  P.output = in->output;
  P.lower = in->lower;
  P.upper = in->upper;
  P.priority = in->priority;
  P.tie_key = in->total_requests > 0 ? in->tie_key : nullptr;
  P.M = static_cast<int32_t>(M);
  return P;
}

sk::Params result_params(const sched_instances_t* in, int64_t M, const sched_results_t* out, int64_t step_cap) {
  sk::Params P = base_params(in, M);
  P.completion = out->completion;
  P.evictions = out->evictions;
  P.total_latency = out->total_latency;
  P.makespan = out->makespan;
  P.request_steps = out->request_steps;
  P.total_evictions = out->total_evictions;
  P.status = out->status;
  P.algo_used = out->algo_used;
  P.step_cap = step_cap;
  return P;
}

// Whether a batch of K instances of at most nmax requests runs a lane per
// instance (k_tiny).  64 instances to a wave last as long as the longest of them, at any K
// up to 262144, while a wave each takes a time that grows with the rounds of 16 waves a
// CU.  Where the two meet depends on how differently long the instances of a wave are.
// From about five rounds on a lane each is ahead or near, but for A_l and A_min of five
// requests or more: promotions and cancellations differ from instance to instance, and A_min
// may cancel hundreds of times where requests are long and the memory is short.  Their
// lines lie between the mixes that suit lanes best and least.  Lane / wave in us,
// (a) the competitive-ratio study's instances (outputs to 6, M = 12), (b) outputs to 512,
// M = 1024, (c) outputs to 32, intervals 1 to 64, M = 96:
//   1 or 2 requests: A_min 11 / 24 for one instance, 24 / 26 for 2048; A_l 33 / 26 for 512,
//     38 / 33 for 8192, 35 / 47 for 16384
//   3 or 4, 20481 instances: A_min 79 / 80, A_l 92 / 80, the others 0.4 to 0.7 of a wave
//   5: A_l 118 / 93 at 20481, 119 / 103 at 24577; A_min (b) 357 / 186, (c) 77 / 89 at 24577
//   6: A_l 150 / 117 at 24577, 149 / 151 at 32768; A_min (a) 139 / 128, (b) 723 / 320 at 24577,
//     155 / 153, 772 / 381 at 32768
//   8: A_l (a) 206 / 140, (c) 73 / 146 at 24577, (a) 212 / 184, (c) 73 / 190 at 32768; A_min (a) 204 /
//     186, (b) 2277 / 989 at 32768, 210 / 259, 2341 / 1402 at 49153, 246 / 633, 2419 / 3310 at 131072;
//     A_random (b) 122 / 79 at 20481, 118 / 90 at 24577, 119 / 158 at 49153; H-SF (a) 91 / 68 at
//     20481, 93 / 97 at 32768; A_max 0.7 to 1.0 of a wave at 20481
// The adaptive policy may run every instance as A_min.
bool tiny_batch(int algo, int64_t nmax, int64_t K, int n_cu) {
  if (nmax > sk::kTinyRequests) return false;
  const bool aell = algo == SCHED_AELL;
  int rounds = 5;
  if (nmax <= 2) rounds = aell ? 3 : 0;
  else if (aell || algo == SCHED_AMIN || algo == SCHED_ADAPTIVE)
    rounds = nmax <= 4 ? 5 : nmax == 5 ? 6 : nmax == 6 || aell ? 8 : 12;
  else if (algo == SCHED_ARANDOM && nmax == 8) rounds = 6;
  return K > rounds * 16 * static_cast<int64_t>(n_cu);
}

const void* tiny_kernel(int algo) {
  switch (algo) {
    case SCHED_AMAX: return reinterpret_cast<const void*>(&sk::k_tiny<SCHED_AMAX>);
    case SCHED_AMIN: return reinterpret_cast<const void*>(&sk::k_tiny<SCHED_AMIN>);
    case SCHED_HSF: return reinterpret_cast<const void*>(&sk::k_tiny<SCHED_HSF>);
    case SCHED_AELL: return reinterpret_cast<const void*>(&sk::k_tiny<SCHED_AELL>);
    case SCHED_ARANDOM: return reinterpret_cast<const void*>(&sk::k_tiny<SCHED_ARANDOM>);
    default: return reinterpret_cast<const void*>(&sk::k_tiny<SCHED_ADAPTIVE>);
  }
}

}  // namespace

extern "C" {

int sched_version(void) { return 131; }

const char* sched_strerror(int code) {
  switch (code) {
    case SCHED_OK: return "ok";
    case SCHED_E_INVAL: return "invalid argument";
    case SCHED_E_INTERVAL: return "invalid request data (o < 1, s < 0, or interval does not contain o)";
    case SCHED_E_TOO_BIG: return "a request can never fit in M";
    case SCHED_E_STEP_CAP: return "step cap reached with unfinished requests";
    case SCHED_E_HIP: return "HIP runtime error";
    case SCHED_E_UNSUPPORTED: return "beyond kernel capacity";
    case SCHED_E_ARRIVAL: return "arrivals negative or not non-decreasing";
    case SCHED_E_SCRATCH: return "workspace beyond the 96 MiB no-allocation scratch";
    default: return "unknown code";
  }
}

int sched_validate(const sched_instances_t* in, int32_t algo, int64_t M, int32_t* status, void* stream) {
  const int c = check_args(in, algo, M);
  if (c != SCHED_OK || in->num_instances == 0) return c;
  if (!status) return SCHED_E_INVAL;
  sk::Params P = base_params(in, M);
  P.status = status;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const dim3 grid(P.K), block(64);
  switch (algo) {
    case SCHED_AMAX: hipLaunchKernelGGL((sk::k_validate<SCHED_AMAX>), grid, block, 0, st, P); break;
    case SCHED_AMIN: hipLaunchKernelGGL((sk::k_validate<SCHED_AMIN>), grid, block, 0, st, P); break;
    case SCHED_HSF: hipLaunchKernelGGL((sk::k_validate<SCHED_HSF>), grid, block, 0, st, P); break;
    case SCHED_AELL: hipLaunchKernelGGL((sk::k_validate<SCHED_AELL>), grid, block, 0, st, P); break;
    case SCHED_ARANDOM: hipLaunchKernelGGL((sk::k_validate<SCHED_ARANDOM>), grid, block, 0, st, P); break;
    default: hipLaunchKernelGGL((sk::k_validate<SCHED_ADAPTIVE>), grid, block, 0, st, P); break;
  }
  return hipGetLastError() == hipSuccess ? SCHED_OK : SCHED_E_HIP;
}

}  // extern "C"

namespace {

// sched_simulate_opts and sched_simulate_noalloc.  no_alloc: the workspace is
// the device's `scratch` array, and the adaptive policy runs both of its
// policies' launches on the caller's stream (no side stream, no events), so
// nothing is allocated.
int simulate_impl(const sched_instances_t* in, int32_t algo, int64_t M, const sched_results_t* out,
                  void* stream, const sched_options_t* opts, bool no_alloc) {
  if (!in || !out) return SCHED_E_INVAL;
  {
    const int c = check_args(in, algo, M);
    if (c != SCHED_OK || in->num_instances == 0) return c;
  }
  if (!out->total_latency || !out->status) return SCHED_E_INVAL;
  if (in->total_requests > 0 && !out->completion) return SCHED_E_INVAL;
  sched_options_t o{};
  if (opts) o = *opts;
  if (o.step_cap > sk::kCapLimit) return SCHED_E_INVAL;
  if (o.running_capacity < 0 || o.evicted_capacity < 0 || o.evicted_lds_limit < 0) return SCHED_E_INVAL;
  if (o.running_capacity > 1024) return SCHED_E_UNSUPPORTED;
  const int ww = o.workgroup_waves <= 1 ? 0 : o.workgroup_waves;
  if (o.workgroup_waves < 0 || (ww != 0 && ww != 2 && ww != 4)) return SCHED_E_INVAL;
  if (ww && (o.running_capacity > 0 || (algo != SCHED_AMAX && algo != SCHED_AMIN && algo != SCHED_HSF)))
    return SCHED_E_INVAL;

  const int64_t nmax = in->max_requests;
  const bool tie = in->total_requests > 0 && in->tie_key != nullptr;
  hipStream_t st = static_cast<hipStream_t>(stream);
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return SCHED_E_HIP;
  int lds_max = 0, n_cu = 0;
  if (hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return SCHED_E_HIP;

  const int nw = static_cast<int>((nmax + 63) / 64);
  const int nw1 = (nw + 63) / 64;
  // LDS: the two bitmap levels, then the cancelled set (8 bytes a slot)
  const size_t lds_bitmaps = 8 * static_cast<size_t>(nw + nw1);
  if (lds_bitmaps + 8 > static_cast<size_t>(lds_max)) return SCHED_E_UNSUPPORTED;
  int cap_fit = static_cast<int>((static_cast<size_t>(lds_max) - lds_bitmaps) / 8);
  if (o.evicted_lds_limit > 0) cap_fit = std::min(cap_fit, o.evicted_lds_limit);
  // the first pass's cancelled-set slots (A_min; A_l's promoted queue is an
  // array of n entries in global memory).  Where many instances share a CU,
  // at most 1024, and for n_max <= 1024 what the LDS share of a wave leaves
  // next to the bitmaps and the staged completion steps (at least 512): an
  // instance whose set outgrows its slots is simulated again by a later pass
  const int64_t waves_cu = std::min<int64_t>(16, std::max<int64_t>(1, (in->num_instances + 255) / 256));
  const int64_t share_room =
      (static_cast<int64_t>(163840 / waves_cu) - 512 - static_cast<int64_t>(lds_bitmaps) - 4 * int64_t(nw) * 64) / 8;
  auto cap0_for = [&](int a) -> int {
    int64_t c = 0;
    if (a == SCHED_AMIN)
      c = std::min<int64_t>(std::max<int64_t>(nmax, 1),
                            in->num_instances <= 64 ? 16384
                            : nmax <= 1024          ? std::min<int64_t>(1024, std::max<int64_t>(512, share_room))
                                                    : 1024);
    if (o.evicted_capacity > 0 && a == SCHED_AMIN) c = o.evicted_capacity;
    return static_cast<int>(std::min<int64_t>(c, cap_fit));
  };
  const int forced_rows = o.running_capacity > 0 ? rows_for(o.running_capacity) : 0;
  // the adaptive policy runs the A_min passes and then the A_l passes; each
  // kernel skips the instances that k_prepare assigned to the other policy
  const int sim_algos[2] = {algo == SCHED_ADAPTIVE ? SCHED_AMIN : static_cast<int>(algo), SCHED_AELL};
  const int n_sim = algo == SCHED_ADAPTIVE ? 2 : 1;
  const Room rm{static_cast<size_t>(lds_max), nw, nw1};
  Tier tiers[2][8];
  int n_tiers[2] = {0, 0};
  bool any_global = algo == SCHED_AELL || algo == SCHED_ADAPTIVE;  // A_l's promoted queue
  // workgroup launches with global cancelled sets: each workgroup simulates
  // its instances one after the other, with n_max entries per wave of its own
  // (at most 64 MiB of them, and at least one workgroup)
  int64_t group_words = 0;
  for (int a = 0; a < n_sim; ++a) {
    n_tiers[a] = build_tiers(sim_algos[a], nmax, in->num_instances, forced_rows, cap0_for(sim_algos[a]), cap_fit,
                             ww, rm, in->num_instances <= 4 * int64_t(n_cu), tiers[a]);
    for (int p = 0; p < n_tiers[a]; ++p) {
      Tier& t = tiers[a][p];
      if (t.gw > 1 && t.vglobal) {
        const int64_t per = static_cast<int64_t>(t.gw) * std::max<int64_t>(nmax, 1);
        t.grid = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(in->num_instances, (int64_t(8) << 20) / per)));
        group_words = std::max<int64_t>(group_words, per * t.grid);
      } else {
        any_global = any_global || t.vglobal;
      }
      // A retry pass takes few of the instances of a large batch, often none, and a
      // workgroup started for each of them costs 200 us at 65536.  A grid that the
      // device holds at once (two or three workgroups a CU) goes through a list of
      // them instead, also where many need it: 65536 instances of which every 4096th,
      // every 256th or one in 20 runs 1200 requests at once, H-SF: 3.2, 5.5 and 17 ms;
      // a workgroup an instance 4.9, 37 and 62 (the device gives workgroups to its XCDs
      // in turn), 4096 workgroups with fixed shares 44, 88 and 148.
      // (After a first launch of workgroups, only A_min instances whose cancelled set is
      // beyond 16384 entries are taken again: fixed shares.)
      if (t.gw > 1 && t.rows == 16 && t.run_mask != 0 && in->num_instances > 16 * int64_t(n_cu)) {
        t.list = 1;
        t.grid = std::min(t.grid > 0 ? t.grid : INT32_MAX, 4 * n_cu);
      }
      if (t.gw > 1 && !sim_kernel_any(sim_algos[a], t)) return SCHED_E_UNSUPPORTED;
    }
  }
  // LDS of a launch before staging (every launch fits, by the choices above)
  auto lds_base = [&](int a, const Tier& t) -> size_t {
    if (t.gw > 1) return group_lds(sim_algos[a], t.gw, t.rows, rm, t.vglobal ? 0 : t.cap_v);
    return lds_bitmaps + (t.vglobal ? 0 : 8 * static_cast<size_t>(t.cap_v));
  };
  for (int a = 0; a < n_sim; ++a)
    for (int p = 0; p < n_tiers[a]; ++p)
      if (lds_base(a, tiers[a][p]) > static_cast<size_t>(lds_max)) return SCHED_E_UNSUPPORTED;

  const size_t N = static_cast<size_t>(in->total_requests);
  const size_t K = static_cast<size_t>(in->num_instances);
  size_t off = 0;
  const size_t o_sa = off; off = align_up(off + 4 * N, 256);
  const size_t o_sb = off; off = align_up(off + 4 * N, 256);
  const size_t o_rec = off; off = align_up(off + 8 * N, 256);
  const size_t o_rk = off; off = align_up(off + 4 * N, 256);
  const size_t o_cap = off; off = align_up(off + 4 * K, 256);
  const size_t o_alg = off; off = align_up(off + (algo == SCHED_ADAPTIVE ? 4 * K : 0), 256);
  const size_t o_tr = off; off = align_up(off + (tie ? 4 * N : 0), 256);
  const size_t o_ix = off; off = align_up(off + (tie ? 4 * N : 0), 256);
  const size_t o_cs = off; off = align_up(off + (tie ? 4 * N : 0), 256);
  const size_t o_es = off; off = align_up(off + (tie && out->evictions ? 4 * N : 0), 256);
  const size_t o_vg = off; off = align_up(off + (any_global ? 8 * N : 0), 256);
  const size_t o_gv = off; off = align_up(off + 8 * static_cast<size_t>(group_words), 256);
  // Priority classes only where every instance of the batch is resident at
  // once (16 waves a CU), so that the launch lasts as long as its slowest
  // instance, and where waves share a SIMD at all (more than one wave on
  // each of a CU's four SIMDs); a batch served in several rounds of waves
  // keeps the priority by unfinished work.
  const bool pcl = (algo == SCHED_AMIN || algo == SCHED_ADAPTIVE) && in->upper != nullptr && in->total_requests > 0 &&
                   static_cast<int64_t>(K) > 4 * static_cast<int64_t>(n_cu) &&
                   static_cast<int64_t>(K) <= 16 * static_cast<int64_t>(n_cu);
  const size_t o_pc = off; off = align_up(off + (pcl ? 4 * K : 0), 256);
  // the launch order of A_min batches that take more than one round of waves
  const bool rounds = static_cast<int64_t>(K) > 16 * static_cast<int64_t>(n_cu);
  const bool ord = algo == SCHED_AMIN && in->total_requests > 0 && rounds;
  const size_t o_or = off; off = align_up(off + (ord ? 8 * K + 4 * sk::kOrderBuckets : 0), 256);
  if (no_alloc && off > kScratchBytes) return SCHED_E_SCRATCH;
  // tiny instances: one launch, a lane each, and no workspace (unless an option
  // asks for a tier of the other kernels)
  if (!ww && forced_rows == 0 && o.evicted_capacity == 0 && o.evicted_lds_limit == 0 &&
      tiny_batch(algo, nmax, in->num_instances, n_cu)) {
    sk::Params P = result_params(in, M, out, o.step_cap);
    hipError_t err = hipSuccess;
    if (o.event_before) err = hipEventRecord(static_cast<hipEvent_t>(o.event_before), st);
    if (err == hipSuccess) {
      const dim3 tgrid((P.K + 63) / 64), tblock(64);
      void* args[] = {&P};
      err = hipLaunchKernel(tiny_kernel(algo), tgrid, tblock, args, 0, st);
    }
    if (err == hipSuccess && o.event_after) err = hipEventRecord(static_cast<hipEvent_t>(o.event_after), st);
    return err == hipSuccess ? SCHED_OK : SCHED_E_HIP;
  }
  // every workspace array is written before it is read (nothing needs clearing)
  void* ws = nullptr;
  if (no_alloc) {
    if (scratch_address(dev, &ws) != hipSuccess) return SCHED_E_HIP;
  } else if (hipMallocAsync(&ws, off + kRetryBytes, st) != hipSuccess) {
    return SCHED_E_HIP;
  }
  char* base = static_cast<char*>(ws);

  sk::Params P = result_params(in, M, out, o.step_cap);
  P.sort_a = reinterpret_cast<uint32_t*>(base + o_sa);
  P.sort_b = reinterpret_cast<uint32_t*>(base + o_sb);
  P.rec = reinterpret_cast<uint2*>(base + o_rec);
  P.rank_of = reinterpret_cast<int32_t*>(base + o_rk);
  P.u_of_rank = reinterpret_cast<int32_t*>(P.sort_b);  // free once the keys are sorted (A_l sorts none)
  P.cap = reinterpret_cast<int32_t*>(base + o_cap);
  P.algo_of = algo == SCHED_ADAPTIVE ? reinterpret_cast<int32_t*>(base + o_alg) : nullptr;
  P.tr_of = tie ? reinterpret_cast<int32_t*>(base + o_tr) : nullptr;
  P.idx_of = tie ? reinterpret_cast<int32_t*>(base + o_ix) : nullptr;
  P.comp_st = tie ? reinterpret_cast<int32_t*>(base + o_cs) : nullptr;
  P.ev_st = tie && out->evictions ? reinterpret_cast<int32_t*>(base + o_es) : nullptr;
  P.vglob = any_global ? reinterpret_cast<uint64_t*>(base + o_vg) : nullptr;
  P.vgroup = group_words ? reinterpret_cast<uint64_t*>(base + o_gv) : nullptr;
  // (only the ladder kernels read the classes and the order)
  const bool ladder = tiers[0][0].grow;
  P.pclass = pcl && ladder ? reinterpret_cast<int32_t*>(base + o_pc) : nullptr;
  P.order = ord && ladder ? reinterpret_cast<int32_t*>(base + o_or) : nullptr;
  P.okey = P.order ? P.order + K : nullptr;
  P.obucket = P.order ? P.okey + K : nullptr;
  int32_t* retry_count = nullptr;
  for (int a = 0; a < n_sim; ++a)
    for (int p = 0; p < n_tiers[a]; ++p)
      if (tiers[a][p].list) retry_count = reinterpret_cast<int32_t*>(base + off);
  P.nw_max = nw;
  P.nw1_max = nw1;
  P.run_cap = forced_rows > 0 ? forced_rows * 64 : INT32_MAX;

  hipError_t err = hipSuccess;
  if (P.order) hipLaunchKernelGGL(sk::k_order_clear, dim3(1), dim3(sk::kOrderBuckets), 0, st, P);
  {
    const PrepareLaunch pl = prepare_launch(algo, nmax, in->num_instances, n_cu, tie, lds_max);
    // (above 64 KiB a kernel's LDS has to be asked for: the buffers and what the kernel
    // itself declares, at most PrepareShared<16>)
    if (pl.lds + sizeof(sk::PrepareShared<16>) > 65536)
      err = hipFuncSetAttribute(pl.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(pl.lds));
    void* args[] = {&P, &retry_count};
    if (err == hipSuccess) err = hipLaunchKernel(pl.kernel, dim3(P.K), dim3(64 * pl.waves), args, pl.lds, st);
    if (pl.spread) hipLaunchKernelGGL(sk::k_spread, dim3(P.K), dim3(64), 0, st);
  }
  if (err == hipSuccess) err = hipGetLastError();
  if (err == hipSuccess && P.pclass) {
    hipLaunchKernelGGL(sk::k_prio_classes, dim3(1), dim3(256), 0, st, P);
    err = hipGetLastError();
  }
  if (err == hipSuccess && P.order) {
    hipLaunchKernelGGL(sk::k_order_scan, dim3(1), dim3(64), 0, st, P);
    hipLaunchKernelGGL(sk::k_order_scatter, dim3((P.K + 255) / 256), dim3(256), 0, st, P);
    err = hipGetLastError();
  }
  // Staging the completion steps in LDS (written out coalesced at the end of
  // an instance instead of one scattered store per completion) when it fits
  // without costing occupancy: at most the LDS share of the waves a CU holds
  // at once (four per SIMD) or that the batch gives it.
  const int64_t nst = static_cast<int64_t>(nw) * 64;
  const int64_t per_cu = std::min<int64_t>(16, std::max<int64_t>(1, (static_cast<int64_t>(K) + 255) / 256));
  const size_t stage_budget = std::min<size_t>(static_cast<size_t>(lds_max), static_cast<size_t>(163840 / per_cu));
  for (int a = 0; a < n_sim; ++a)
    for (int p = 0; p < n_tiers[a]; ++p) {
      Tier& t = tiers[a][p];
      t.stage = 0;
      // (a workgroup launch: when it fits at all; few instances run at once)
      if (lds_base(a, t) + 4 * nst <= (t.gw > 1 ? static_cast<size_t>(lds_max) : stage_budget)) t.stage = 1;
    }
  auto lds_of = [&](int a, const Tier& t) -> size_t { return lds_base(a, t) + (t.stage ? 4 * nst : 0); };
  for (int a = 0; a < n_sim && err == hipSuccess; ++a)
    for (int p = 0; p < n_tiers[a] && err == hipSuccess; ++p)
      if (lds_of(a, tiers[a][p]) > 65536)
        err = hipFuncSetAttribute(sim_kernel_any(sim_algos[a], tiers[a][p], P.order && tiers[a][p].grid <= 0,
                                                 P.pclass != nullptr, rounds),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_of(a, tiers[a][p])));
  if (err == hipSuccess && o.event_before) err = hipEventRecord(static_cast<hipEvent_t>(o.event_before), st);
  // adaptive: the A_l launches go to the side stream after the preparation,
  // and the caller's stream waits for them before the end (fork and join)
  hipStream_t side = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  if (err == hipSuccess && n_sim == 2 && !no_alloc) {
    err = side_stream(dev, &side);
    if (err == hipSuccess) err = hipEventCreateWithFlags(&fork, hipEventDisableTiming);
    if (err == hipSuccess) err = hipEventCreateWithFlags(&join, hipEventDisableTiming);
    if (err == hipSuccess) err = hipEventRecord(fork, st);
    if (err == hipSuccess) err = hipStreamWaitEvent(side, fork, 0);
  }
  for (int a = 0; a < n_sim && err == hipSuccess; ++a) {
    const hipStream_t sa = a == 1 && side ? side : st;
    for (int p = 0; p < n_tiers[a] && err == hipSuccess; ++p) {
      const Tier& t = tiers[a][p];
      sk::Params q = P;
      q.cap_v = t.cap_v;
      q.retry_status = t.rows_status;
      q.retry_v_status = t.v_status;
      q.run_mask = t.run_mask;
      q.stage_comp = t.stage;
      sk::RetryList rl{};
      if (t.list) {
        // (the sort buffer is free now and has room for them: every listed instance has
        // more than 640 requests, of its own unless offsets decrease; the adaptive
        // policy's two passes run at the same time)
        rl.list = reinterpret_cast<int32_t*>(P.sort_a) + (a == 1 ? N / 2 : 0);
        rl.room = static_cast<int32_t>(std::min<size_t>(n_sim == 2 ? N / 2 : N, INT32_MAX));
        rl.count = retry_count + 2 * (8 * a + p);
        hipLaunchKernelGGL(sk::k_retry_list, dim3((P.K + 255) / 256), dim3(256), 0, sa, q, rl, sim_algos[a]);
        err = hipGetLastError();
      }
      void* args[] = {&q, &rl};  // (the list: its kernels alone)
      const dim3 tgrid(t.grid > 0 ? t.grid : P.K), tblock(64 * (t.gw > 1 ? t.gw : 1));
      // (a launch over every instance may take them in the launch order)
      if (err == hipSuccess)
        err = hipLaunchKernel(sim_kernel_any(sim_algos[a], t, P.order && t.grid <= 0, P.pclass != nullptr, rounds),
                              tgrid, tblock, args, lds_of(a, t), sa);
    }
  }
  if (side) {
    // join even after a failed launch, so that the workspace is not freed
    // while work queued on the side stream may still use it
    hipError_t je = join ? hipEventRecord(join, side) : hipErrorInvalidValue;
    if (je == hipSuccess) je = hipStreamWaitEvent(st, join, 0);
    if (je != hipSuccess) je = hipStreamSynchronize(side);
    if (err == hipSuccess) err = je;
  }
  if (fork) (void)hipEventDestroy(fork);
  if (join) (void)hipEventDestroy(join);
  if (err == hipSuccess && o.event_after) err = hipEventRecord(static_cast<hipEvent_t>(o.event_after), st);
  const hipError_t ferr = no_alloc ? hipSuccess : hipFreeAsync(ws, st);
  if (err != hipSuccess || ferr != hipSuccess) return SCHED_E_HIP;
  return SCHED_OK;
}

}  // namespace

extern "C" {

int sched_simulate_opts(const sched_instances_t* in, int32_t algo, int64_t M,
                        const sched_results_t* out, void* stream, const sched_options_t* opts) {
  return simulate_impl(in, algo, M, out, stream, opts, false);
}

int sched_simulate_noalloc(const sched_instances_t* in, int32_t algo, int64_t M,
                           const sched_results_t* out, void* stream, const sched_options_t* opts) {
  return simulate_impl(in, algo, M, out, stream, opts, true);
}

int sched_simulate(const sched_instances_t* in, int32_t algo, int64_t M,
                   const sched_results_t* out, void* stream) {
  return sched_simulate_opts(in, algo, M, out, stream, nullptr);
}

}  // extern "C"
