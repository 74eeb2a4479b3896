// Shared by the PFACT leaf kernels: argmax reductions and the tagged-word
// exchange between the workgroups of a leaf (protocol in panel_leaf.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>

#include "common.h"
#include "kernels.h"

namespace {

// (value, index) argmax: larger value wins, equal values go to the smaller
// index (the first maximum, as in BLAS idamax).  NaN never wins.
__device__ __forceinline__ void argmax_merge(double &v, int &idx, double ov, int oidx) {
    if (ov > v || (ov == v && oidx < idx)) {
        v = ov;
        idx = oidx;
    }
}

__device__ __forceinline__ void wave_argmax(double &v, int &idx) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double ov = __shfl_xor(v, off);
        const int oi = __shfl_xor(idx, off);
        argmax_merge(v, idx, ov, oi);
    }
}

constexpr int kRowWords = 2 * mxlu::kLeafW;      // a leaf row, two words per value
constexpr int kSlotWords = 4 + kRowWords;

__device__ __forceinline__ void ll_store(uint64_t *p, uint32_t seq, uint32_t payload) {
    __hip_atomic_store(p, ((uint64_t)seq << 32) | payload, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t ll_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Bounded waiting, after `spins` looks: true when the caller has to give up.  Once
// any wait has expired the results are invalid: later waits give up at their
// first check (every `period` looks) instead of spinning.
__device__ __forceinline__ bool ll_give_up(int spins, int limit, int period, int *flags) {
    if (spins >= limit) {
        atomicExch(&flags[1], 1);
        return true;
    }
    return (spins & (period - 1)) == period - 1 &&
           __hip_atomic_load(&flags[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// Payload of *p once it carries `seq`; x is a load of *p already issued.
__device__ __forceinline__ uint32_t ll_wait(const uint64_t *p, uint64_t x, uint32_t seq, int limit,
                                           int *flags) {
    for (int spins = 0; (uint32_t)(x >> 32) != seq; ++spins) {
        if (ll_give_up(spins, limit, 1024, flags)) break;
        __builtin_amdgcn_s_sleep(1);
        x = ll_load(p);
    }
    return (uint32_t)x;
}

// Wait until each word x[k] with bit k of `valid` carries `seq` (x holds
// loads already issued; addr(k) is the word's address).  Every round re-issues
// the loads of all words still stale at once, so a round costs one load
// latency however many words are late; the loop is wave-uniform.
template <int K, class Addr>
__device__ __forceinline__ void ll_gather(uint64_t (&x)[K], uint32_t valid, Addr addr, uint32_t seq,
                                          int limit, int *flags) {
    for (int rounds = 0;; ++rounds) {
        uint32_t stale = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (((valid >> k) & 1u) && (uint32_t)(x[k] >> 32) != seq) stale |= 1u << k;
        if (__builtin_amdgcn_ballot_w64(stale != 0) == 0) break;
        if (ll_give_up(rounds, limit, 64, flags)) break;
        __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if ((stale >> k) & 1u) x[k] = ll_load(addr(k));
    }
}

template <int CTRL>
__device__ __forceinline__ void argmax_dpp(double &v, int &idx) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
    const int oi = __builtin_amdgcn_update_dpp(0, idx, CTRL, 0xF, 0xF, false);
    argmax_merge(v, idx,
                 __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo)), oi);
}

// every lane ends with the wave's (max, first index); all lanes active
__device__ __forceinline__ void wave_argmax_dpp(double &v, int &idx) {
    argmax_dpp<0xB1>(v, idx);    // quad_perm [1,0,3,2]
    argmax_dpp<0x4E>(v, idx);    // quad_perm [2,3,0,1]
    argmax_dpp<0x124>(v, idx);   // row_ror:4
    argmax_dpp<0x128>(v, idx);   // row_ror:8 (each row of 16 lanes now agrees)
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    double rv = -1.0;
    int ri = INT_MAX;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 16 * r);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 16 * r);
        argmax_merge(rv, ri, __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)),
                     __builtin_amdgcn_readlane(idx, 16 * r));
    }
    v = rv;
    idx = ri;
}

}  // namespace
