// prepare.hpp -- what runs before the simulation (device code of k_validate and
// k_prepare): an instance's checks, its initial outputs and its ranked records.
//
// A workgroup of W waves takes one instance.  What bounds it: 2000 requests of
// 65536 instances are 2.6 GB in and out (0.5 ms), but a stable radix pass is a chain of
// LDS round trips, one per 64 elements of a wave, and the sort buffers (8 bytes a
// request) leave a CU room for few workgroups, so one wave each kept 10 waves on a
// CU and its chains' latency showed.  Hence W waves share an instance's buffers, each
// with a histogram and a stretch of the elements of its own, the arrays are read
// once (checks, sums, initial outputs and sort keys come from the same pass), and a
// sort covers only the bits in which the keys differ, in as few passes of at most
// eight bits as that takes, of equal width (each bit is one ballot an element).
// Measured (one wave an instance, every key byte sorted, the arrays read two to four
// times -> now): 65536 x 2000 H-SF 3.46 -> 1.45 ms, 3000 x 1500 with tie keys 242 -> 87 us,
// 1024 x 10000 A_min 850 -> 273 us, one A_max instance of 100000 3.58 -> 0.38 ms.
#pragma once

#include "sim_device.hpp"

namespace sk {

template <int W>
struct PrepareShared {
  alignas(16) uint32_t hist[W * 256];
  int64_t sums[W][4];
  uint32_t bits[W][3];
};

// A barrier of the workgroup's waves; one wave alone orders its LDS accesses by
// issuing them.
template <int W>
__device__ __forceinline__ void prepare_sync() {
  if (W > 1) __syncthreads();
  else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// One stable LSD radix pass over the n elements src[0..n) -> dst by the digit
// (key(element) >> shift) of `bits` <= 8 bits: every wave counts the digits of its
// stretch of the elements, finds where each of them goes (after the smaller digits
// and the earlier waves'), and scatters its stretch 64 elements at a time, equal
// digits ranked by one ballot a bit.
template <int W, typename KeyFn>
__device__ __forceinline__ void radix_pass(PrepareShared<W>& sh, const uint32_t* src, uint32_t* dst, int n, int shift,
                                           int bits, KeyFn key) {
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int w = wave::uniform(static_cast<int>(threadIdx.x) >> 6);
  uint32_t* const hist = sh.hist + 256 * w;
  const uint32_t mask = (1u << bits) - 1u;
  const int per = ((n + W - 1) / W + 63) & ~63;
  const int lo = w * per, hi = lo + per < n ? lo + per : n;
  reinterpret_cast<uint4*>(hist)[lane] = make_uint4(0, 0, 0, 0);
  prepare_sync<1>();
  for (int i = lo + lane; i < hi; i += 64) atomicAdd(&hist[(key(src[i]) >> shift) & mask], 1u);
  prepare_sync<W>();
  {
    // digits 4 * lane to 4 * lane + 3: all waves' counts, and the earlier waves'
    uint4 all = make_uint4(0, 0, 0, 0), before = all;
#pragma unroll
    for (int v = 0; v < W; ++v) {
      const uint4 h = reinterpret_cast<const uint4*>(sh.hist + 256 * v)[lane];
      all.x += h.x; all.y += h.y; all.z += h.z; all.w += h.w;
      if (v < w) {
        before.x += h.x; before.y += h.y; before.z += h.z; before.w += h.w;
      }
    }
    const uint32_t tot = all.x + all.y + all.z + all.w;
    const uint32_t ex = static_cast<uint32_t>(wave::inclusive_scan_i32(static_cast<int32_t>(tot))) - tot;
    prepare_sync<W>();
    reinterpret_cast<uint4*>(hist)[lane] = make_uint4(ex + before.x, ex + all.x + before.y, ex + all.x + all.y + before.z,
                                                      ex + all.x + all.y + all.z + before.w);
  }
  prepare_sync<1>();
  const uint64_t lt_mask = lane == 0 ? 0ull : ~0ull >> (64 - lane);
  for (int c = lo; c < hi; c += 64) {
    const int i = c + lane;
    const bool act = i < hi;
    const uint32_t e = act ? src[i] : 0u;
    const uint32_t d = act ? (key(e) >> shift) & mask : 0u;
    uint64_t eq = wave::ballot(act);
    for (int bit = 0; bit < bits; ++bit) {
      const uint64_t bal = wave::ballot((d >> bit) & 1u);
      eq &= ((d >> bit) & 1u) ? bal : ~bal;
    }
    if (act) {
      const int rank = __builtin_popcountll(eq & lt_mask);
      const uint32_t base = hist[d];
      dst[base + rank] = e;
      prepare_sync<1>();  // every lane has read its digit's counter
      if (rank == 0) hist[d] = base + static_cast<uint32_t>(__builtin_popcountll(eq));
    }
    prepare_sync<1>();
  }
  prepare_sync<W>();
}

// Stable sort of the n elements of a by the 32-bit key(element), which differ in
// the bits `varies` only; b: a second buffer.  Returns the one with the result.
template <int W, typename KeyFn>
__device__ __forceinline__ uint32_t* radix_sort(PrepareShared<W>& sh, uint32_t* a, uint32_t* b, int n, uint32_t varies,
                                                KeyFn key) {
  while (varies != 0u) {
    const int shift = __builtin_ctz(varies);
    const int span = 32 - __builtin_clz(varies) - shift;
    const int passes = (span + 7) / 8;
    const int bits = (span + passes - 1) / passes;
    radix_pass<W>(sh, a, b, n, shift, bits, key);
    varies &= ~(((1u << bits) - 1u) << shift);
    uint32_t* const t = a;
    a = b;
    b = t;
  }
  return a;
}

// The bits in which the keys of the workgroup's lanes differ, from each lane's
// conjunction and disjunction of the keys it has seen.
template <int W>
__device__ __forceinline__ uint32_t varying_bits(PrepareShared<W>& sh, uint32_t kand, uint32_t kor) {
  for (int off = 32; off >= 1; off >>= 1) {
    kand &= static_cast<uint32_t>(__shfl_xor(static_cast<int>(kand), off, 64));
    kor |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(kor), off, 64));
  }
  if (W > 1) {
    const int w = static_cast<int>(threadIdx.x) >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
      sh.bits[w][0] = kand;
      sh.bits[w][1] = kor;
    }
    __syncthreads();
    for (int v = 0; v < W; ++v) {
      kand &= sh.bits[v][0];
      kor |= sh.bits[v][1];
    }
  }
  return wave::uniform_u(kand ^ kor);
}

// What an instance's requests add up to.
struct Checked {
  int status, algo, n;      // n: requests of an instance whose offsets are sound, else 0
  int64_t cap;              // step cap
  int64_t sum_o, sum_l, sum_u;   // of o, and of the bounds that were read
};

// Checks instance k (shared by k_prepare and k_validate): the status, the policy
// the instance runs (the adaptive choice) and the default step cap.  WIDTHS: the
// sums of both bounds are wanted.  each(i, o, lower, upper, priority) is called for every
// request of an instance whose offsets are sound, with the bounds that the policy reads.
template <int ALGO, int W, typename EachFn>
__device__ __forceinline__ Checked check_instance(const Params& P, PrepareShared<W>& sh, int k, bool widths, EachFn each) {
  const int64_t b = P.offsets[k];
  const int64_t e = P.offsets[k + 1];
  Checked r;
  r.status = (b < 0 || e < b || e > P.N || e - b > P.max_requests) ? SCHED_E_INVAL : SCHED_OK;
  r.n = r.status == SCHED_OK ? static_cast<int>(e - b) : 0;

  // l is read by A_min and A_l, u by A_max and A_l; the adaptive policy reads
  // both (their sums pick the policy) and validates with the one it picks
  constexpr bool kReadL = ALGO == SCHED_AMIN || ALGO == SCHED_AELL || ALGO == SCHED_ADAPTIVE;
  constexpr bool kReadU = ALGO == SCHED_AMAX || ALGO == SCHED_AELL || ALGO == SCHED_ADAPTIVE;
  constexpr bool kReadP = ALGO == SCHED_ARANDOM;
  enum { kArr = 1, kInt = 2, kBig = 4, kUnsup = 8, kBadL = 16, kUnsupL = 32, kBadU = 64, kBigU = 128, kUnsupU = 256 };
  uint32_t bad = r.n >= (1 << kIdxBits) ? kUnsup : 0;
  int32_t max_a = 0;
  int64_t sum_o = 0, sum_l = 0, sum_u = 0;
  for (int i = threadIdx.x; i < r.n; i += 64 * W) {
    const int32_t a = P.arrival ? P.arrival[b + i] : 0;
    const int32_t ap = P.arrival && i > 0 ? P.arrival[b + i - 1] : 0;
    const int32_t s = P.prompt[b + i];
    const int32_t o = P.output[b + i];
    const int32_t lo = kReadL ? P.lower[b + i] : 1;
    const int32_t up = kReadU || widths ? P.upper[b + i] : 1;
    const int32_t pr = kReadP ? P.priority[b + i] : 0;
    if (a < 0 || (i > 0 && a < ap)) bad |= kArr;
    if (o < 1 || s < 0) bad |= kInt;
    if (lo < 1 || lo > o) bad |= kBadL;
    if (up < o) bad |= kBadU;
    if (static_cast<int64_t>(s) + o > P.M) bad |= kBig;
    if (static_cast<int64_t>(s) + up > P.M) bad |= kBigU;
    if (o >= kEstLimit || s >= kPromptLimit || pr < 0 || pr >= kEstLimit) bad |= kUnsup;
    if (lo >= kEstLimit) bad |= kUnsupL;
    if (up >= kEstLimit) bad |= kUnsupU;
    max_a = a > max_a ? a : max_a;
    sum_o += o;
    sum_l += lo;
    sum_u += up;
    each(i, o, lo, up, pr);
  }
  sum_o = wave::sum_i64(sum_o);
  if (kReadL) sum_l = wave::sum_i64(sum_l);
  if (kReadU || widths) sum_u = wave::sum_i64(sum_u);
  for (int off = 32; off >= 1; off >>= 1) {
    bad |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(bad), off, 64));
    const int32_t m = __shfl_xor(max_a, off, 64);
    max_a = m > max_a ? m : max_a;
  }
  if (W > 1) {
    const int w = static_cast<int>(threadIdx.x) >> 6;
    if ((threadIdx.x & 63) == 0) {
      sh.sums[w][0] = sum_o;
      sh.sums[w][1] = sum_l;
      sh.sums[w][2] = sum_u;
      sh.sums[w][3] = max_a;
      sh.bits[w][2] = bad;
    }
    __syncthreads();
    sum_o = sum_l = sum_u = 0;
    for (int v = 0; v < W; ++v) {
      sum_o += sh.sums[v][0];
      sum_l += sh.sums[v][1];
      sum_u += sh.sums[v][2];
      max_a = sh.sums[v][3] > max_a ? static_cast<int32_t>(sh.sums[v][3]) : max_a;
      bad |= sh.bits[v][2];
    }
  }
  // the policy this instance runs; the adaptive one takes A_l when
  // L/U < (3 - sqrt 5)/2, i.e. sqrt(5) U < 3U - 2L, i.e. 5U^2 < (3U - 2L)^2
  r.algo = ALGO;
  if (ALGO == SCHED_ADAPTIVE) {
    const int64_t d = 3 * sum_u - 2 * sum_l;
    r.algo = SCHED_AMIN;
    if (r.n > 0 && d > 0) {
      const unsigned __int128 dd = static_cast<unsigned __int128>(d) * static_cast<unsigned __int128>(d);
      const unsigned __int128 uu = static_cast<unsigned __int128>(sum_u) * static_cast<unsigned __int128>(sum_u);
      if (dd > 5 * uu) r.algo = SCHED_AELL;
    }
  }
  const bool use_l = r.algo == SCHED_AMIN || r.algo == SCHED_AELL;
  const bool use_u = r.algo == SCHED_AMAX || r.algo == SCHED_AELL;
  if (r.status == SCHED_OK) {
    if (bad & kArr) r.status = SCHED_E_ARRIVAL;
    else if (bad & (kInt | (use_l ? kBadL : 0) | (use_u ? kBadU : 0))) r.status = SCHED_E_INTERVAL;
    else if (bad & (kBig | (use_u ? kBigU : 0))) r.status = SCHED_E_TOO_BIG;
    else if (bad & (kUnsup | (use_l ? kUnsupL : 0) | (use_u ? kUnsupU : 0))) r.status = SCHED_E_UNSUPPORTED;
  }
  int64_t cap = P.step_cap > 0 ? P.step_cap : 4 * (max_a + sum_o + r.n) + 64;
  r.cap = cap > kCapLimit ? kCapLimit : cap;
  r.sum_o = sum_o;
  r.sum_l = sum_l;
  r.sum_u = sum_u;
  return r;
}

// Validation only (sched_validate): status per instance.
template <int ALGO>
__global__ __launch_bounds__(64) void k_validate(Params P) {
  __shared__ PrepareShared<1> sh;
  const int k = blockIdx.x;
  const Checked r = check_instance<ALGO>(P, sh, k, false, [](int, int32_t, int32_t, int32_t, int32_t) {});
  if (threadIdx.x == 0) {
    P.status[k] = r.status;
    if (P.algo_used) P.algo_used[k] = r.algo;
  }
}

// LDS: the sort buffers of max_requests entries are in LDS (with tie keys a third
// one holds these), else in the workspace.  retry_count: the retry passes' counts, to be
// cleared (or NULL).
template <int ALGO, int W, bool LDS>
__global__ __launch_bounds__(64 * W) void k_prepare(Params P, int32_t* retry_count) {
  __shared__ PrepareShared<W> sh;
  extern __shared__ uint32_t pre_buf[];
  constexpr int kStride = 64 * W;
  const int k = blockIdx.x;
  const int tid = static_cast<int>(threadIdx.x);
  const int64_t b = P.offsets[k];
  const bool tie = P.tie_key != nullptr;
  uint32_t* const ka = LDS ? pre_buf : P.sort_a + b;
  uint32_t* const kb = LDS ? pre_buf + P.max_requests : P.sort_b + b;
  if (retry_count && k == 0 && tid < kRetryCounts) retry_count[tid] = 0;

  // ---- checks; per-request outputs start as "not completed, never cancelled"
  // (with tie keys, the staging arrays the kernels write too); without tie keys,
  // the keys (k0 << 17 | index), k0 = u (A_max), l (A_min, A_l), o (H-SF), the
  // priority (A_random, which plans with o)
  uint32_t kand = 0xFFFFFFFFu, kor = 0u;
  const auto start_value = [&](int32_t o, int32_t lo, int32_t up, int32_t pr) {
    return static_cast<uint32_t>(ALGO == SCHED_AMAX ? up : ALGO == SCHED_HSF ? o : ALGO == SCHED_ARANDOM ? pr : lo);
  };
  const Checked r = check_instance<ALGO>(P, sh, k, P.pclass != nullptr,
                                         [&](int i, int32_t o, int32_t lo, int32_t up, int32_t pr) {
    P.completion[b + i] = -1;
    if (P.evictions) P.evictions[b + i] = 0;
    if (tie) {
      P.comp_st[b + i] = -1;
      if (P.evictions) P.ev_st[b + i] = 0;
    }
    const uint32_t est = start_value(o, lo, up, pr);
    kand &= est;
    kor |= est;
    if (!tie) ka[i] = (est << kIdxBits) | static_cast<uint32_t>(i);
  });
  const int algo = r.algo;
  const int n = r.status == SCHED_OK ? r.n : 0;
  if (tid == 0) {
    P.status[k] = r.status;
    P.cap[k] = static_cast<int32_t>(r.cap);
    if (P.algo_of) P.algo_of[k] = algo;
    if (P.algo_used) P.algo_used[k] = algo;
    // wide intervals mean more cancellations, so longer simulations: the
    // class by sum(u - l) / sum(l) (< 0.3, < 0.75, above)
    if (P.pclass) {
      const int64_t w = r.sum_u - r.sum_l;
      P.pclass[k] = n == 0 || algo != SCHED_AMIN ? 3 : 4 * w >= 3 * r.sum_l ? 2 : 10 * w >= 3 * r.sum_l ? 1 : 0;
    }
    if (P.okey) {
      // A_min cancels until its lower bounds have grown to the true lengths, so
      // the instances whose lower bounds fall furthest below them run longest:
      // the key is 16 * sum(o - l) / sum(l), at most kOrderBuckets - 1
      const int64_t q = n > 0 && r.sum_l > 0 ? (16 * (r.sum_o - r.sum_l)) / r.sum_l : 0;
      const int key = q < kOrderBuckets - 1 ? static_cast<int>(q) : kOrderBuckets - 1;
      P.okey[k] = key;
      atomicAdd(&P.obucket[key], 1);
    }
  }
  if (n == 0) return;
  uint32_t varies = varying_bits(sh, kand, kor);

  uint32_t* src = ka;
  uint32_t* other = kb;
  if (tie) {
    // ---- tie keys: each request's rank in the order (tie key, index) (A_l:
    // (arrival, tie key, index), its fresh-queue order) is its identity in the
    // keys; tr_of maps index -> rank, idx_of rank -> index
    const int32_t* const tk = P.tie_key + b;
    uint32_t* const tv = pre_buf + 2 * P.max_requests;  // (LDS)
    const auto tie_bits = [&](uint32_t i) { return LDS ? tv[i] : static_cast<uint32_t>(tk[i]) ^ 0x80000000u; };
    uint32_t tand = 0xFFFFFFFFu, tor = 0u;
    for (int i = tid; i < n; i += kStride) {
      const uint32_t v = static_cast<uint32_t>(tk[i]) ^ 0x80000000u;
      ka[i] = static_cast<uint32_t>(i);
      if (LDS) tv[i] = v;
      tand &= v;
      tor |= v;
    }
    const uint32_t tvary = varying_bits(sh, tand, tor);
    prepare_sync<W>();
    src = radix_sort<W>(sh, ka, kb, n, tvary, tie_bits);
    if (algo == SCHED_AELL && P.arrival) {
      // (arrivals are not negative, and the last one is the latest)
      const int32_t* const ar = P.arrival + b;
      const uint32_t last = static_cast<uint32_t>(ar[n - 1]);
      src = radix_sort<W>(sh, src, src == ka ? kb : ka, n, last == 0u ? 0u : 0xFFFFFFFFu >> __builtin_clz(last),
                          [&](uint32_t i) { return static_cast<uint32_t>(ar[i]); });
    }
    other = src == ka ? kb : ka;
    for (int q = tid; q < n; q += kStride) {
      const uint32_t i = src[q];
      P.tr_of[b + i] = q;
      P.idx_of[b + q] = static_cast<int32_t>(i);
      const int32_t est = algo == SCHED_AMAX ? P.upper[b + i] : algo == SCHED_HSF ? P.output[b + i]
                          : algo == SCHED_ARANDOM ? P.priority[b + i] : P.lower[b + i];
      other[q] = (static_cast<uint32_t>(est) << kIdxBits) | static_cast<uint32_t>(q);
    }
    uint32_t* const t = src;
    src = other;
    other = t;
  }
  prepare_sync<W>();
  // (A_l's queue is in id order: its ranks are the ids, no sort)
  if (algo != SCHED_AELL) src = radix_sort<W>(sh, src, other, n, varies, [](uint32_t key) { return key >> kIdxBits; });
  // ---- ranked records and inverse ranks (rank_of is indexed by request index,
  // and read only where some request arrives after step 0)
  const bool late = late_arrivals(P, b, n);
  for (int q = tid; q < n; q += kStride) {
    const uint32_t key = src[q];
    const uint32_t id = key & kIdxMask;
    const uint32_t idx = tie ? static_cast<uint32_t>(P.idx_of[b + id]) : id;
    const uint32_t s = static_cast<uint32_t>(P.prompt[b + idx]);
    const uint32_t o = static_cast<uint32_t>(P.output[b + idx]);
    P.rec[b + q] = make_uint2(key, s | (o << 16));
    if (late) P.rank_of[b + idx] = q;
    if (algo == SCHED_AELL) P.u_of_rank[b + q] = P.upper[b + idx];
  }
}

}  // namespace sk
