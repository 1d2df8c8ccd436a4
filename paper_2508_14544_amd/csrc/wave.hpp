// wave.hpp -- wave64 primitives for gfx950 (CDNA4).
//
// 32-bit reductions that go to a scalar register (max_i32, sum_i32, min_u32) fold by
// DPP alone into lane 63, row shifts and then row broadcasts (fold_to_last).  Those
// that leave the result in every lane (sum_i32_all, sum4_i32, min_u32_all) first fold
// the four 16-lane rows onto each other with the gfx950 lane swaps
// (v_permlane32_swap, v_permlane16_swap), then run a DPP butterfly inside each row
// (quad_perm 1,0,3,2 / 2,3,0,1, row_half_mirror, row_mirror).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace wave {

constexpr int kDppQuadXor1 = 0xB1;    // quad_perm [1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;    // quad_perm [2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;
constexpr int kDppWaveShl1 = 0x130;  // lane i reads lane i + 1
constexpr int kDppWaveShr1 = 0x138;  // lane i reads lane i - 1

__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__device__ __forceinline__ int32_t readlane(int32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

__device__ __forceinline__ uint32_t readlane_u(uint32_t v, int lane) {
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int32_t>(v), lane));
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
  uint32_t lo = readlane_u(static_cast<uint32_t>(v), lane);
  uint32_t hi = readlane_u(static_cast<uint32_t>(v >> 32), lane);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// v_writelane_b32 through its LLVM intrinsic (this compiler has no clang builtin
// for it): the compiler knows its semantics and inserts the wait states.
extern "C" __device__ int32_t sk_llvm_writelane(int32_t src, int32_t lane, int32_t old)
    __asm("llvm.amdgcn.writelane");

// v with lane `lane` replaced by the uniform value s (the other lanes keep v)
__device__ __forceinline__ int32_t writelane(int32_t v, int32_t s, int lane) {
  return sk_llvm_writelane(s, lane, v);
}

__device__ __forceinline__ uint32_t writelane_u(uint32_t v, uint32_t s, int lane) {
  return static_cast<uint32_t>(writelane(static_cast<int32_t>(v), static_cast<int32_t>(s), lane));
}

__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uniform_u(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int32_t>(v)));
}

// The same value, held in vector registers: the compiler treats the result
// as varying per lane.  For wave-uniform state that is used rarely (array
// base addresses, counters), so that it does not take scalar registers
// through the hot loops; loads and stores take vector addresses anyway.
template <typename T>
__device__ __forceinline__ T in_vgpr(T v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The same value, opaque to the compiler and in a scalar register: for a uniform
// value that would otherwise be drawn into vector code (a constant that a vector
// instruction of the same block uses too, a chain of minima that becomes one
// three-operand vector minimum), which would take every branch on it along.
__device__ __forceinline__ int32_t in_sgpr(int32_t v) {
  v = __builtin_amdgcn_readfirstlane(v);  // (no instruction where it is in one already)
#ifdef __OPTIMIZE__
  asm("" : "+s"(v));
#endif
  return v;
}

// (every control used reads some lane for every lane, or leaves the rest to
// the caller, so the old value does not matter)
template <int CTRL>
__device__ __forceinline__ int32_t dpp(int32_t v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}

// Cross-row folds (gfx950): after fold_rows every lane holds OP over the four
// lanes {l mod 16 + 16 k}; v_permlane32_swap exchanges the two 32-lane halves
// and v_permlane16_swap the odd and even 16-lane rows.
template <typename F>
__device__ __forceinline__ uint32_t fold_rows(uint32_t v, F op) {
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = op(static_cast<uint32_t>(h[0]), static_cast<uint32_t>(h[1]));
  const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return op(static_cast<uint32_t>(q[0]), static_cast<uint32_t>(q[1]));
}

template <typename F>
__device__ __forceinline__ uint32_t fold_in_row(uint32_t v, F op) {
  v = op(v, static_cast<uint32_t>(dpp<kDppQuadXor1>(static_cast<int32_t>(v))));
  v = op(v, static_cast<uint32_t>(dpp<kDppQuadXor2>(static_cast<int32_t>(v))));
  v = op(v, static_cast<uint32_t>(dpp<kDppRowHalfMirror>(static_cast<int32_t>(v))));
  v = op(v, static_cast<uint32_t>(dpp<kDppRowMirror>(static_cast<int32_t>(v))));
  return v;
}

struct OpMaxI32 {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const {
    return static_cast<int32_t>(a) > static_cast<int32_t>(b) ? a : b;
  }
};
struct OpAddU32 {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; }
};
struct OpMinU32 {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a < b ? a : b; }
};

// The fold left in lane 63 only: inside each row by row_shr 1, 2, 4, 8, then
// from row to row by row_bcast 15 and 31, one instruction a step (a lane without
// a source folds `none`, the identity, which the hardware does by not writing
// it).  12 instructions with their wait states, where folding the rows with lane
// swaps first takes 17: for results that go to a scalar register at once.
template <uint32_t NONE, typename F>
__device__ __forceinline__ uint32_t fold_to_last(uint32_t v, F op) {
  auto step = [&](auto ctrl, auto rows) {
    v = op(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(static_cast<int32_t>(NONE), static_cast<int32_t>(v),
                                                                decltype(ctrl)::value, decltype(rows)::value, 0xF, false)));
  };
  step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});
  step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});
  step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});
  step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});
  step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});
  step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});
  return v;
}

__device__ __forceinline__ int32_t max_i32(int32_t v) {
  return readlane(static_cast<int32_t>(fold_to_last<0x80000000u>(static_cast<uint32_t>(v), OpMaxI32{})), 63);
}

__device__ __forceinline__ int32_t sum_i32(int32_t v) {
  return readlane(static_cast<int32_t>(fold_to_last<0u>(static_cast<uint32_t>(v), OpAddU32{})), 63);
}

// The sum left in every lane (a vector value): for tests that combine it with
// other per-lane conditions before a single ballot.
__device__ __forceinline__ int32_t sum_i32_all(int32_t v) {
  return static_cast<int32_t>(fold_in_row(fold_rows(static_cast<uint32_t>(v), OpAddU32{}), OpAddU32{}));
}

// Four sums at once: lanes 16 q to 16 q + 15 get the sum of vq over the wave.
// The lane swaps put two half-folded values into one register, so the four
// share one in-row fold: 10 instructions where four sums of their own take 32.
__device__ __forceinline__ int32_t sum4_i32(int32_t v0, int32_t v1, int32_t v2, int32_t v3) {
  const auto a = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(v0), static_cast<uint32_t>(v2), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(v1), static_cast<uint32_t>(v3), false, false);
  const uint32_t s02 = static_cast<uint32_t>(a[0]) + static_cast<uint32_t>(a[1]);
  const uint32_t s13 = static_cast<uint32_t>(b[0]) + static_cast<uint32_t>(b[1]);
  const auto q = __builtin_amdgcn_permlane16_swap(s02, s13, false, false);
  return static_cast<int32_t>(fold_in_row(static_cast<uint32_t>(q[0]) + static_cast<uint32_t>(q[1]), OpAddU32{}));
}

// The minimum left in every lane, for locating it with a ballot without a
// round trip through a scalar register.
__device__ __forceinline__ uint32_t min_u32_all(uint32_t v) { return fold_in_row(fold_rows(v, OpMinU32{}), OpMinU32{}); }

__device__ __forceinline__ uint32_t min_u32(uint32_t v) {
  return readlane_u(fold_to_last<0xFFFFFFFFu>(v, OpMinU32{}), 63);
}

// Stores and atomics of the lanes in `mask`, for code that a whole wave runs
// with every lane active (exec is all ones before and after).  A branch on the
// lane would do the same, but one such branch inside a loop makes the compiler
// rebuild the loop's whole control flow out of condition masks (it only leaves
// regions alone whose branches are all uniform); with these, a loop whose
// other branches are uniform keeps plain scalar branches.  The compiler does not
// count these operations: its own waits for later loads still hold (the counters
// are in order, so an extra operation only makes them stricter), and code that
// reads the stored values from global memory waits with wait_stores first (LDS
// operations of a wave are executed in order).
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)(p)));
}
#ifdef __OPTIMIZE__
__device__ __forceinline__ void lds_store32(uint64_t mask, uint32_t at, uint32_t v) {
  asm volatile("s_mov_b64 exec, %0\n\tds_write_b32 %1, %2\n\ts_mov_b64 exec, -1" ::"s"(mask), "v"(at), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_store64(uint64_t mask, uint32_t at, uint64_t v) {
  asm volatile("s_mov_b64 exec, %0\n\tds_write_b64 %1, %2\n\ts_mov_b64 exec, -1" ::"s"(mask), "v"(at), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_or64(uint64_t mask, uint32_t at, uint64_t v) {
  asm volatile("s_mov_b64 exec, %0\n\tds_or_b64 %1, %2\n\ts_mov_b64 exec, -1" ::"s"(mask), "v"(at), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_and64(uint64_t mask, uint32_t at, uint64_t v) {
  asm volatile("s_mov_b64 exec, %0\n\tds_and_b64 %1, %2\n\ts_mov_b64 exec, -1" ::"s"(mask), "v"(at), "v"(v) : "memory");
}
__device__ __forceinline__ void global_store32(uint64_t mask, const void* at, uint32_t v) {
  asm volatile("s_mov_b64 exec, %0\n\tglobal_store_dword %1, %2, off\n\ts_mov_b64 exec, -1" ::"s"(mask), "v"(at), "v"(v)
               : "memory");
}
__device__ __forceinline__ void global_store64(uint64_t mask, const void* at, uint64_t v) {
  asm volatile("s_mov_b64 exec, %0\n\tglobal_store_dwordx2 %1, %2, off\n\ts_mov_b64 exec, -1" ::"s"(mask), "v"(at), "v"(v)
               : "memory");
}
// (device scope: the counts are in the L2 that every CU of the XCD shares, as a
// plain agent-scope fetch-add without a result)
__device__ __forceinline__ void global_add32(uint64_t mask, const void* at, uint32_t v) {
  asm volatile("s_mov_b64 exec, %0\n\tglobal_atomic_add %1, %2, off\n\ts_mov_b64 exec, -1" ::"s"(mask), "v"(at), "v"(v)
               : "memory");
}
#else
// (without optimisation a uniform value need not be in a scalar register: there
// the branch on the lane it is)
__device__ __forceinline__ bool in_mask(uint64_t mask) { return (mask >> lane_id()) & 1ull; }
template <typename T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds_at(uint32_t at) {
  return (__attribute__((address_space(3))) T*)(static_cast<uintptr_t>(at));
}
__device__ __forceinline__ void lds_store32(uint64_t mask, uint32_t at, uint32_t v) {
  if (in_mask(mask)) *lds_at<uint32_t>(at) = v;
}
__device__ __forceinline__ void lds_store64(uint64_t mask, uint32_t at, uint64_t v) {
  if (in_mask(mask)) *lds_at<uint64_t>(at) = v;
}
__device__ __forceinline__ void lds_or64(uint64_t mask, uint32_t at, uint64_t v) {
  if (in_mask(mask)) __hip_atomic_fetch_or(lds_at<uint64_t>(at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_and64(uint64_t mask, uint32_t at, uint64_t v) {
  if (in_mask(mask)) __hip_atomic_fetch_and(lds_at<uint64_t>(at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void global_store32(uint64_t mask, const void* at, uint32_t v) {
  if (in_mask(mask)) *static_cast<uint32_t*>(const_cast<void*>(at)) = v;
}
__device__ __forceinline__ void global_store64(uint64_t mask, const void* at, uint64_t v) {
  if (in_mask(mask)) *static_cast<uint64_t*>(const_cast<void*>(at)) = v;
}
__device__ __forceinline__ void global_add32(uint64_t mask, const void* at, uint32_t v) {
  if (in_mask(mask))
    __hip_atomic_fetch_add(static_cast<uint32_t*>(const_cast<void*>(at)), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
#endif
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// 64-bit sums for the epilogue (not on the hot path).
__device__ __forceinline__ int64_t sum_i64(int64_t v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ int64_t max_i64(int64_t v) {
  for (int off = 32; off >= 1; off >>= 1) {
    int64_t o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  return v;
}

// Inclusive prefix sum over the wave (setup only).
__device__ __forceinline__ int32_t inclusive_scan_i32(int32_t v) {
  const int lane = lane_id();
  for (int off = 1; off < 64; off <<= 1) {
    int32_t o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  return v;
}

}  // namespace wave
