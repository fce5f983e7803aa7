// Device side of the one-launch periods (PeriodArgs in launch.h): values that
// travel between running workgroups as (value, epoch) pairs.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch.h"

namespace cmcg {

// A pair is 8 bytes -- 32 value bits below a 32-bit epoch -- written and read
// by one aligned 8-byte access of agent scope, so a reader that finds the
// epoch it waits for has the value with it: no flag, no fence, and one
// memory round trip between a store and its reader.  FP64 values take two
// pairs (low word, high word).
template <typename T> struct Tagged;

template <> struct Tagged<float> {
    static constexpr int W = 1;
    typedef unsigned long long In;
    static __device__ __forceinline__ void put(unsigned long long* p, float v, uint32_t epoch) {
        __hip_atomic_store(p, (unsigned long long)__float_as_uint(v) | ((unsigned long long)epoch << 32),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ void get(const unsigned long long* p, In& w) {
        w = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ bool ok(In w, uint32_t epoch) { return (uint32_t)(w >> 32) == epoch; }
    static __device__ __forceinline__ float value(In w) { return __uint_as_float((uint32_t)w); }
};

template <> struct Tagged<double> {
    static constexpr int W = 2;
    struct In {
        unsigned long long lo, hi;
    };
    static __device__ __forceinline__ void put(unsigned long long* p, double v, uint32_t epoch) {
        const unsigned long long u = (unsigned long long)__double_as_longlong(v);
        const unsigned long long e = (unsigned long long)epoch << 32;
        __hip_atomic_store(p, (u & 0xffffffffull) | e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p + 1, (u >> 32) | e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ void get(const unsigned long long* p, In& w) {
        w.lo = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        w.hi = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ bool ok(const In& w, uint32_t epoch) {
        return (uint32_t)(w.lo >> 32) == epoch && (uint32_t)(w.hi >> 32) == epoch;
    }
    static __device__ __forceinline__ double value(const In& w) {
        return __longlong_as_double((long long)((w.lo & 0xffffffffull) | (w.hi << 32)));
    }
};

// Called after a poll that found a pair missing (spin = polls so far, t0 = 0
// at the wait's start): true when the wave has to give up, because the wait
// has passed the time limit or another workgroup has given up.  Every wait
// ends: a workgroup whose neighbours never run (they found no room on the
// device) marks the launch failed, and the host runs the period by stage
// launches instead.
__device__ __forceinline__ bool period_stuck(const PeriodArgs& a, uint32_t spin, unsigned long long& t0) {
    if ((spin & 63u) != 63u) return false;
    const unsigned long long t = wall_clock64();
    if (t0 == 0) t0 = t;
    if (__hip_atomic_load(a.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.epoch) return true;
    if (t - t0 <= a.limit) return false;
    __hip_atomic_store(a.abort, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return true;
}

// The inbox of a workgroup: n contiguous values (n uniform over the
// workgroup) that its neighbours write for this epoch.  request() asks for the
// first R values per thread, settle() waits until every value has arrived --
// the rest in batches of R -- and hands value i to take(i, r, v), r its place in
// the first batch or R.  settle() returns false when the wave gave up.
template <typename T, int R, int NTH> struct Inbox {
    using X = Tagged<T>;
    typename X::In w[R];
    __device__ __forceinline__ void request(const unsigned long long* in, int first, int n, int tid) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = first + tid + NTH * r;
            if (i < n) X::get(in + (uint32_t)i * X::W, w[r]);
        }
    }
    // the batch requested from `first` on; r = a value's place in it
    template <typename F>
    __device__ __forceinline__ bool settle_batch(const unsigned long long* in, int first, int n, int tid,
                                                 uint32_t epoch, const PeriodArgs& a, F take) {
        unsigned long long t0 = 0;
        for (uint32_t spin = 0;; ++spin) {
            bool ok = true;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = first + tid + NTH * r;
                if (i < n && !X::ok(w[r], epoch)) {
                    ok = false;
                    X::get(in + (uint32_t)i * X::W, w[r]);
                }
            }
            if (__all(ok)) break;
            if (period_stuck(a, spin, t0)) return false;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = first + tid + NTH * r;
            if (i < n) take(i, r, X::value(w[r]));
        }
        return true;
    }
    template <typename F>
    __device__ __forceinline__ bool settle(const unsigned long long* in, int n, int tid, uint32_t epoch,
                                           const PeriodArgs& a, F take) {
        for (int first = 0; first < n; first += NTH * R) {
            if (first > 0) request(in, first, n, tid);
            if (!settle_batch(in, first, n, tid, epoch, a, [&](int i, int r, T v) { take(i, first == 0 ? r : R, v); }))
                return false;
        }
        return true;
    }
};

// Workgroups of a period kernel that the device holds at once: what the
// occupancy query allows.  Blocks whose waves do not divide over the four SIMDs
// of a compute unit need a free wave slot besides: with five slots per SIMD, four
// blocks of five waves were not placed (799 blocks of k_period_col<3> waited in
// vain), three were, and six blocks of three waves.
template <typename F> inline int64_t resident_room(F kernel, int threads) {
    int dev = 0, cus = 0, fit = 0;
    CMCG_HIP(hipGetDevice(&dev));
    CMCG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    CMCG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, kernel, threads, 0));
    const int waves = threads / 64;
    if (waves % 4 != 0) {
        hipFuncAttributes at;
        CMCG_HIP(hipFuncGetAttributes(&at, reinterpret_cast<const void*>(kernel)));
        const int slots = 512 / ((at.numRegs + 7) / 8 * 8);  // per SIMD, at most 8
        const int limit = (4 * (slots < 8 ? slots : 8) - 1) / waves;
        if (fit > limit) fit = limit;
    }
    return (int64_t)fit * cus;
}

// Launches a period kernel over nblocks element blocks and n members (those of
// a.order from a.first on).
template <typename F>
inline void launch_resident(F kernel, int64_t nblocks, int n, int left_out, int threads, const PeriodArgs& a,
                            hipStream_t s) {
    const int64_t per = (nblocks + 7) / 8;
    const dim3 grid((unsigned)(8 * (per - left_out)), (unsigned)n);
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, a, per);
    CMCG_HIP(hipGetLastError());
}

}  // namespace cmcg
