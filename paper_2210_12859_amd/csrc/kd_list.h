// kd_list.h -- device helpers shared by the traversal kernels: wave votes,
// result keys, the sorted k-best list and record loads.
#pragma once

#include <hip/hip_runtime.h>

#include "kd_internal.h"

namespace kd {

namespace {

constexpr uint32_t SENT_IDX = 0x7fffffffu;  // index word of an empty list slot

// Wave votes on a lane predicate held as a lane mask (no round trip through
// a VGPR, as the int-argument forms take).
__device__ __forceinline__ uint64_t wave_ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool wave_any(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// Between LDS writes of some lanes of a wave and reads of the same memory by
// others.  The wave's LDS instructions are done in order, so this only holds the
// compiler to that order; it costs no instruction.
__device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__device__ __forceinline__ uint64_t make_key(float d2, int32_t idx) {
    return (uint64_t(__float_as_uint(d2)) << 32) | uint32_t(idx);
}

__device__ __forceinline__ float key_d2(uint64_t key) { return __uint_as_float(uint32_t(key >> 32)); }

// 64-bit keys as doubles: the bit patterns of non-negative doubles order like
// unsigned integers, and no key reaches the exponent of infinity (the high
// word is at most that of a binary32 infinity), so v_min_f64 / v_max_f64 take
// the smaller / larger key in one instruction each (denormal patterns pass
// unchanged).
__device__ __forceinline__ uint64_t key_min(uint64_t a, uint64_t b) {
    uint64_t r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ uint64_t key_max(uint64_t a, uint64_t b) {
    uint64_t r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Sorted insertion of `key` into the ascending list L (its largest key drops
// out; a key above it changes nothing): slot j becomes key clamped to
// [L[j-1], L[j]], two instructions.  The network runs for the whole wave
// whenever a lane inserts, and the step kernels are bound by vector
// instructions; against the median of the high words plus a 64-bit compare
// and two selects (four instructions a slot), calls of 1M 3-D queries: k = 8
// 0.721 -> 0.691 ms, with split planes only 0.712 -> 0.659 ms; 150K 2-D
// queries, k = 50: 0.885 -> 0.666 ms.
template <int K>
__device__ __forceinline__ void list_insert(uint64_t (&L)[K], uint64_t key) {
    if constexpr (K == 1) {
        L[0] = key < L[0] ? key : L[0];
        return;
    }
#pragma unroll
    for (int j = K - 1; j > 0; --j) L[j] = key_max(L[j - 1], key_min(key, L[j]));
    L[0] = key_min(key, L[0]);
}

}  // namespace

}  // namespace kd
