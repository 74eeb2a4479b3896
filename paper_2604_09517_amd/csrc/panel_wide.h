// PFACT leaf, wide form (FP64 and FP32, leaves of any width up to 32 columns,
// up to kWideMaxGroups workgroups): the column steps, pivot choice and
// arithmetic of the forms in panel_leaf.hip, bit for bit, on the fewest
// workgroups that hold the rows in registers: NT threads with RPT rows each
// (1024 rows, which fill a CU's registers in FP64).
//
// What bounds a leaf is the chain of dependent latencies of each column, so
// everything is chosen to shorten that chain:
//   * rows never move between threads: every thread keeps the position its
//     row has in the interchanged panel, an interchange exchanges two
//     positions, and each row is stored to its position at the end (after
//     every workgroup has loaded its rows).
//   * up to 1024 rows: one workgroup, no exchange through memory at all, one
//     LDS barrier per column: every wave leaves its candidate (value,
//     position, row) in LDS, after the barrier every wave picks the winner.
//   * more rows: one exchange round trip per column instead of two.  The
//     group's candidate row goes out together with its position, and every
//     group reads all candidates' rows in one batch (each wave reads every
//     NT/64-th group's row, one word per lane), so no second, dependent read
//     of the winner's row follows.  With 1024 rows per group that batch is
//     at most 32 KB per group and column; 256-row groups would make it four
//     times that for four times the readers.
// The columns are unrolled eight at a time: after each eight the row's
// registers are renamed by a rotation (register c then holds column
// (8 jb + c) % 32), which keeps every register index a constant without
// unrolling all 32 columns (eight minutes of compilation instead of one).
// The wave reduction takes the maximum of the upper words by DPP and finds
// its lane by ballot; only ties in the upper word take the full comparison.
//
// Measured per 32-column FP64 leaf on an MI355X, in brackets the 256-row
// register form it replaced: 256 rows 44 us (123), 1024 rows 60 us (124),
// 4096 rows 123 us (132), 16384 rows 136 us (145), 32768 rows 150 us (160).
// Of a column's 1.2 us in one workgroup about a third is the two candidate
// reductions, a third the candidate rows' way through LDS; with an exchange
// about 1.2 us are the store-to-load latency between XCDs (a bare exchange
// among 2 to 32 workgroups takes 1.0 to 1.5 us).
#pragma once

#include "common.h"
#include "panel_exchange.h"

namespace {

// (v, idx) of the first maximum over the wave; idx is the tie-break, v = -1
// marks a lane without a candidate.  Uniform results.
__device__ __forceinline__ void wave_first_max(double &v, int &idx) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)(b >> 32);
    // v is -1 or >= 0, so the upper words order as signed integers
    int mx = hi;
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x124, 0xF, 0xF, false));   // row_ror:4
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x128, 0xF, 0xF, false));   // row_ror:8
    const int m0 = max(__builtin_amdgcn_readlane(mx, 0), __builtin_amdgcn_readlane(mx, 16));
    const int m1 = max(__builtin_amdgcn_readlane(mx, 32), __builtin_amdgcn_readlane(mx, 48));
    const int top = max(m0, m1);
    // no candidate: at most one lane of the leaf still has a position (row J)
    const uint64_t at = top < 0 ? __builtin_amdgcn_ballot_w64(idx != INT_MAX)
                                : __builtin_amdgcn_ballot_w64(hi == top);
    if (__builtin_popcountll(at) <= 1) {
        const int l = at ? __builtin_ctzll(at) : 0;
        const uint32_t rl = (uint32_t)__builtin_amdgcn_readlane(lo, l);
        const uint32_t rh = (uint32_t)__builtin_amdgcn_readlane(hi, l);
        v = __longlong_as_double((long long)(((uint64_t)rh << 32) | rl));
        idx = __builtin_amdgcn_readlane(idx, l);
    } else {
        wave_argmax_dpp(v, idx);
    }
}

template <typename T, int NT>
struct WideShared {
    static constexpr int NW = NT / 64;
    // the waves' candidates, by parity of the column: without an exchange a
    // column's data is read until the next column's only barrier
    double cv[2][NW];
    int ci[2][NW];
    __attribute__((aligned(16))) T crow[2][NW][mxlu::kLeafW];
    // exchange: the waves' winners over the groups they read
    double gv[NW];
    int gi[NW];
    __attribute__((aligned(16))) T grow[NW][mxlu::kLeafW];
};

// EXCH: the leaf may span several workgroups
template <typename T, int NT, int RPT, bool EXCH>
struct WideLeaf {
    static constexpr int W = mxlu::kLeafW, NW = NT / 64, R = NT * RPT;
    static constexpr int CB = 8, NB = W / CB;                // columns per unrolled block
    static constexpr int VW = (int)sizeof(T) / 4;            // 32-bit words of a value
    static constexpr int RW = W * VW;                        // ... of a row
    static constexpr int KR = (mxlu::kWideMaxGroups + NW - 1) / NW;   // groups read per wave
    T x[RPT][W];     // register c: column (CB jb + c) % W in block jb
    int pos[RPT];    // the row's position in the interchanged leaf (-1: no row)
    int m, w, G, g, tid, lane, wave;
    int64_t r0;
    int32_t *ipiv;
    uint64_t *slots;
    int *flags;

    // (v, idx) of the wave's entry with index `lane`, reduced to the first
    // maximum; returns the lane it came from
    __device__ __forceinline__ int pick(double &v, int &idx) {
        const int mine = idx;
        wave_first_max(v, idx);
        const uint64_t at = __builtin_amdgcn_ballot_w64(mine == idx && lane < NW);
        return at ? __builtin_ctzll(at) : 0;
    }

    template <int JL>
    __device__ __forceinline__ void column(WideShared<T, NT> &sh, int jb) {
        const int J = CB * jb + JL, par = JL & 1;
        const uint32_t seq = (uint32_t)(r0 + J + 1);
        // the wave's candidate: first position >= J of largest |x| (NaN never
        // wins; position J itself is the choice when nothing else is)
        double v = -1.0;
        int idx = INT_MAX;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            if (pos[q] == J && idx == INT_MAX) idx = J;
            const double av = fabs((double)x[q][JL]);
            if (pos[q] >= J && (av > v || (av == v && pos[q] < idx))) {
                v = av;
                idx = pos[q];
            }
        }
        wave_first_max(v, idx);
        T *cand = &sh.crow[par][wave][0];
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            if (pos[q] == idx) {   // its row, from column CB jb on (zeros before)
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    if (RPT > 1 && k >= NB - jb) break;   // uniform
                    T *d = cand + CB * ((jb + k) % NB);
#pragma unroll
                    for (int c = 0; c < CB; ++c) d[c] = k < NB - jb ? x[q][CB * k + c] : (T)0;
                }
            }
        if (lane == 0) {
            sh.cv[par][wave] = v;
            sh.ci[par][wave] = idx;
        }
        lds_barrier();
        v = lane < NW ? sh.cv[par][lane] : -1.0;
        idx = lane < NW ? sh.ci[par][lane] : INT_MAX;
        const T *prow = nullptr;
        T piv, un;
        auto lane_value = [&](T t, int l) -> T {   // uniform: lane l's t
            if constexpr (sizeof(T) == 8) {
                const uint64_t b = (uint64_t)__double_as_longlong(t);
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
                const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
                return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
            } else {
                return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), l));
            }
        };
        const int JN = J + 1 < W ? J + 1 : J, ln = lane < NW ? lane : 0;
        if (!EXCH || G == 1) {
            // values J and J + 1 of every candidate row come in the same LDS
            // round as the candidates themselves
            const T pl = sh.crow[par][ln][J], ul = sh.crow[par][ln][JN];
            const int from = pick(v, idx);
            prow = &sh.crow[par][from][0];
            piv = lane_value(pl, from);
            un = lane_value(ul, from);
        } else if constexpr (EXCH) {
            const int own = pick(v, idx);
            uint64_t *gs = slots + (size_t)par * mxlu::kMaxGroups * kSlotWords;
            const int first = VW * CB * jb;   // first word in use
            if (wave == own) {   // the wave that holds the row
                const uint32_t *words = reinterpret_cast<const uint32_t *>(&sh.crow[par][wave][0]);
                uint64_t *mine = gs + (size_t)g * kSlotWords;
                if (lane >= first && lane < RW) ll_store(&mine[4 + lane], seq, words[lane]);
                if (lane == 0) ll_store(&mine[2], seq, (uint32_t)idx);
            }
            // one batch: rows of groups wave, wave + NW, ... (a word per lane)
            // and their positions (lane k: the k-th of them); words not read
            // count as arrived
            const int cnt = wave < G ? (G - wave + NW - 1) / NW : 0;
            const bool rd = lane >= first && lane < RW;
            const uint64_t *pr = gs + (size_t)wave * kSlotWords + 4 + lane;
            const uint64_t *pi = gs + (size_t)(wave + NW * (lane < cnt ? lane : 0)) * kSlotWords + 2;
            const uint64_t none = (uint64_t)seq << 32;
            uint64_t xw[KR], xi = none;
            auto stale = [&](uint64_t t) { return (uint32_t)(t >> 32) != seq; };
#pragma unroll
            for (int k = 0; k < KR; ++k)
                xw[k] = k < cnt && rd ? ll_load(pr + k * (NW * kSlotWords)) : none;
            if (lane < cnt) xi = ll_load(pi);
            for (long rounds = 0;; ++rounds) {
                bool late = stale(xi);
#pragma unroll
                for (int k = 0; k < KR; ++k) late = late || stale(xw[k]);
                if (__builtin_amdgcn_ballot_w64(late) == 0) break;
                if ((rounds & 63) == 63) {
                    // once any wait has expired the results are invalid:
                    // later waits give up at their first check
                    if (__hip_atomic_load(&flags[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                        break;
                    if (rounds > (1L << 22)) {
                        atomicExch(&flags[1], 1);
                        break;
                    }
                }
                __builtin_amdgcn_s_sleep(1);
#pragma unroll
                for (int k = 0; k < KR; ++k)
                    if (stale(xw[k])) xw[k] = ll_load(pr + k * (NW * kSlotWords));
                if (stale(xi)) xi = ll_load(pi);
            }
            double bv = -1.0;
            int bi = INT_MAX;
            uint32_t bw = 0;
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                if (k < cnt) {   // wave-uniform
                    const int ki = __builtin_amdgcn_readlane((int)(uint32_t)xi, k);
                    double kv;
                    if (sizeof(T) == 8) {
                        const uint32_t a =
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)xw[k], (2 * J) & 63);
                        const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)xw[k],
                                                                               (2 * J + 1) & 63);
                        kv = fabs(__longlong_as_double((long long)(((uint64_t)b << 32) | a)));
                    } else {
                        kv = fabs((double)__int_as_float(
                            __builtin_amdgcn_readlane((int)(uint32_t)xw[k], J)));
                    }
                    if (ki == INT_MAX || !(kv >= 0.0)) kv = -1.0;   // none, or a NaN at J
                    if (kv > bv || (kv == bv && ki < bi)) {
                        bv = kv;
                        bi = ki;
                        bw = (uint32_t)xw[k];
                    }
                }
            }
            if (lane < RW) reinterpret_cast<uint32_t *>(sh.grow[wave])[lane] = bw;
            if (lane == 0) {
                sh.gv[wave] = bv;
                sh.gi[wave] = bi;
            }
            lds_barrier();
            v = lane < NW ? sh.gv[lane] : -1.0;
            idx = lane < NW ? sh.gi[lane] : INT_MAX;
            const T pl = sh.grow[ln][J], ul = sh.grow[ln][JN];
            const int from = pick(v, idx);
            prow = &sh.grow[from][0];
            piv = lane_value(pl, from);
            un = lane_value(ul, from);
        }
        // the pivot row's values, on their way while the multipliers are formed
        T u[W];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const T *src = prow + CB * ((jb + k) % NB);
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (CB * k + c > JL + 1) u[CB * k + c] = src[c];
        }
        // a position outside [J, m) can only follow an expired wait (stale
        // words): position J then, so no index leaves the panel
        int p = idx;
        if (p < J || p >= m) p = J;
        const bool nonzero = v != 0.0;
        if (!nonzero) p = J;   // an exactly zero column is left as it is
        if (g == 0 && tid == 0) {
            ipiv[J] = (int32_t)(r0 + p);
            if (!nonzero && flags[0] == 0) flags[0] = (int)(r0 + J + 1);
        }
        constexpr int CN = JL + 1 < W ? JL + 1 : JL;
        T l[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            pos[q] = pos[q] == p ? J : (pos[q] == J ? p : pos[q]);
            l[q] = nonzero ? x[q][JL] / piv : x[q][JL];
        }
        // rows up to position J are final: not even a multiple by zero, which
        // an infinity in the pivot row would turn into NaN
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            if (pos[q] > J) {
                x[q][JL] = l[q];
                if (JL + 1 < CB || jb + 1 < NB) x[q][CN] = fma(-l[q], un, x[q][CN]);
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    // one row per thread: finished columns take 0 * 0 (exact);
                    // two: they are skipped (uniform)
                    if (RPT > 1 && k >= NB - jb) break;
                    const T lk = k == 0 || k < NB - jb ? l[q] : (T)0;
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        if (CB * k + c > JL + 1)
                            x[q][CB * k + c] = fma(-lk, u[CB * k + c], x[q][CB * k + c]);
                }
            }
    }

    template <int JL>
    __device__ __forceinline__ void block(WideShared<T, NT> &sh, int jb) {
        if constexpr (JL < CB) {
            if (CB * jb + JL < w) {   // uniform
                column<JL>(sh, jb);
                block<JL + 1>(sh, jb);
            }
        }
    }

    __device__ __forceinline__ void rotate() {
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            T t[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) t[c] = x[q][c];
#pragma unroll
            for (int c = 0; c < W - CB; ++c) x[q][c] = x[q][c + CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) x[q][W - CB + c] = t[c];
        }
    }
};

template <typename T, int NT, int RPT, bool EXCH>
__global__ __launch_bounds__(NT) void panel_leaf_wide_kernel(int m, int w, T *__restrict__ P,
                                                             int64_t lda, int G, int64_t r0,
                                                             int32_t *__restrict__ ipiv,
                                                             uint64_t *slots, int *flags) {
    __shared__ WideShared<T, NT> sh;
    using Leaf = WideLeaf<T, NT, RPT, EXCH>;
    Leaf s;
    s.m = m;
    s.w = w;
    s.G = G;
    s.g = blockIdx.x;
    s.tid = threadIdx.x;
    s.lane = s.tid & 63;
    s.wave = __builtin_amdgcn_readfirstlane(s.tid >> 6);
    s.r0 = r0;
    s.ipiv = ipiv;
    s.slots = slots;
    s.flags = flags;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = s.g * Leaf::R + s.tid + NT * q;
        s.pos[q] = r < m ? r : -1;
#pragma unroll
        for (int c = 0; c < Leaf::W; ++c)
            s.x[q][c] = (r < m && c < w) ? P[(size_t)r + (size_t)c * lda] : (T)0;
    }
    for (int jb = 0; jb < Leaf::NB; ++jb) {
        s.template block<0>(sh, jb);
        s.rotate();   // four rotations bring the columns back to their registers
    }
    // a row may go to another group's position: every group has loaded its
    // rows before the first exchange (or barrier) of the leaf completed
#pragma unroll
    for (int q = 0; q < RPT; ++q)
        if (s.pos[q] >= 0) {
#pragma unroll
            for (int c = 0; c < Leaf::W; ++c)
                if (c < w) P[(size_t)s.pos[q] + (size_t)c * lda] = s.x[q][c];
        }
}

}  // namespace

namespace mxlu {

template <typename T>
int panel_leaf_wide(int64_t m, int w, T *P, int64_t ldp, int64_t r0, int32_t *ipiv, int G,
                    const PanelExchange &ex, hipStream_t s) {
    if (m <= 0 || w <= 0 || w > kLeafW || G > kWideMaxGroups || (int64_t)G * 1024 < m) {
        set_error_msg("panel_leaf_wide: bad shape");
        return MXLU_E_NOMEM;
    }
    // up to 256 rows: four waves with a row per thread (fewer waves meet at
    // each barrier and read the pivot row)
    if (m <= 256)
        hipLaunchKernelGGL((panel_leaf_wide_kernel<T, 256, 1, false>), dim3(1), dim3(256), 0, s,
                           (int)m, w, P, ldp, 1, r0, ipiv + r0, ex.slots, ex.flags);
    else
        hipLaunchKernelGGL((panel_leaf_wide_kernel<T, 512, 2, true>), dim3((unsigned)G), dim3(512),
                           0, s, (int)m, w, P, ldp, G, r0, ipiv + r0, ex.slots, ex.flags);
    MXLU_LAUNCH_CHECK();
    return 0;
}

}  // namespace mxlu
