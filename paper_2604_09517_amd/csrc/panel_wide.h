// PFACT leaf, wide form (FP64 and FP32, leaves of any width up to 32 columns,
// up to kWideMaxGroups workgroups): the column steps, pivot choice and
// arithmetic of the forms in panel_leaf.hip, bit for bit, on the fewest
// workgroups that hold the rows in registers: NT threads with RPT rows each, of
// which CW columns are held at a time.
//
// What bounds a leaf is the chain of dependent latencies of each column, so
// everything is chosen to shorten that chain:
//   * rows never move between threads: every thread keeps the position its
//     row has in the interchanged leaf, an interchange exchanges two
//     positions, and rows are stored to their positions (after every
//     workgroup has loaded that part of its rows).
//   * one row per thread where one workgroup holds them so, up to four else:
//     the reductions and bookkeeping of a column are issued once per wave, an
//     instruction every four cycles, whatever the rows of a lane.  Four rows
//     of 32 FP64 columns do not fit a thread's vector registers, so that such
//     a leaf is taken in two halves of 16 columns: the second is loaded when
//     the first is done, takes the first's columns (its 16 pivot rows'
//     triangular solve, then one product per thread and row) and is factored
//     like the first.  The first half's columns are left to the caller's
//     interchanges for those of the second half (panel_leaf_swap).
//   * no load is under a condition, and rows are updated four columns a masked
//     region.
//   * up to 2048 rows: one workgroup, no exchange through memory.  Two LDS
//     barriers per column: the waves' candidates (value, position) meet in
//     LDS, every wave picks the winner and divides while the winner's wave
//     writes its row.
//   * more rows: one exchange round trip per column.  The group's candidate
//     row goes out with its position; every wave reads all groups' candidates
//     (a lane per group) and picks the winner itself, and in the same batch
//     its share of the rows, so that no second, dependent read of the winner's
//     row follows.
//   * the columns are unrolled four at a time: after each four the row's
//     registers are renamed by a rotation, which keeps every register index a
//     constant.  Unrolled by 32 or by eight the code is executed once or a few
//     times a leaf, does not fit the instruction cache, and every step waits
//     for the instruction fetch.
// The wave reduction takes the maximum of the upper words by DPP and finds
// its lane by ballot; only ties in the upper word take the full comparison.
//
// A leaf of 32 FP64 columns with 64 / 256 / 512 / 1024 / 1500 / 2048 / 4096 /
// 8192 / 16384 / 32768 rows takes 22 / 31 / 37 / 53 / 67 / 72 / 91 / 98 / 120 /
// 145 us.  All in halves above 256 rows and with an exchange from 1025 rows on it
// was 35 / 36 / 54 / 58 / 124 / 124 / 130 / 132 / 132 / 149; as 32 workgroups or
// more with two exchange rounds per column 123 us up to 4096 rows, 145 and 160
// us.  The interchanges that follow take 5.8 us in one launch; composing and
// applying them in two took 12 to 16 us.
#pragma once

#include "common.h"
#include "panel_exchange.h"

namespace {

// Maximum over the wave (uniform).
__device__ __forceinline__ int wave_max_i32(int mx) {
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x124, 0xF, 0xF, false));   // row_ror:4
    mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x128, 0xF, 0xF, false));   // row_ror:8
    const int a = max(__builtin_amdgcn_readlane(mx, 0), __builtin_amdgcn_readlane(mx, 16));
    const int b = max(__builtin_amdgcn_readlane(mx, 32), __builtin_amdgcn_readlane(mx, 48));
    return max(a, b);
}

// The upper word of |x| (all of it in FP32), -1 for NaN: orders candidates up
// to ties.
__device__ __forceinline__ int cand_key(double x) {
    const int h = (int)((uint64_t)__double_as_longlong(x) >> 32) & 0x7fffffff;
    return x == x ? h : -1;
}
__device__ __forceinline__ int cand_key(float x) {
    return x == x ? __float_as_int(x) & 0x7fffffff : -1;
}

// The lane (uniform) of the first maximum of v, ties by index (every lane
// takes part; rarely needed).
__device__ __forceinline__ int first_of(double v, int idx) {
    const double v0 = v;
    const int i0 = idx;
    wave_argmax_dpp(v, idx);
    return __builtin_ctzll(__builtin_amdgcn_ballot_w64(v0 == v && i0 == idx));
}

struct __attribute__((aligned(16))) WideKey {
    double v;   // the candidate's value
    int idx;    // its position (INT_MAX: no candidate)
    int key;    // its key; -1: no candidate but the stand-in at position J
};

template <typename T, int NT, int CW>
struct WideShared {
    static constexpr int NW = NT / 64;
    WideKey cand[NW];   // the waves' candidates
    // the pivot row and the group's candidate row to publish (unfinished
    // blocks of columns only)
    __attribute__((aligned(16))) T row[CW];
    __attribute__((aligned(16))) T stage[CW];
    // halves: rows of the first half's pivots (their multipliers), and the
    // same rows of the second half
    __attribute__((aligned(16))) T l11[CW][CW];
    __attribute__((aligned(16))) T u12[CW][CW];
};

// CW columns of a leaf at a time (CW < 32: two halves).  EXCH: the leaf may
// span several workgroups.
template <typename T, int NT, int RPT, int CW, bool EXCH>
struct WideLeaf {
    static constexpr int NW = NT / 64, R = NT * RPT;
    static constexpr int CB = 4, NB = CW / CB;               // columns per unrolled block
    static constexpr int VW = (int)sizeof(T) / 4;            // 32-bit words of a value
    static constexpr int RW = CW * VW;                       // ... of a row
    static constexpr int GPL = 64 / (RW < 64 ? RW : 64);     // groups' rows per wave load
    static constexpr int KR = (mxlu::kWideMaxGroups + NW * GPL - 1) / (NW * GPL);
    T x[RPT][CW];    // register c: column (CB jb + c) % CW of the half in block jb
    int pos[RPT];    // the row's position in the interchanged leaf (-1: no row)
    int m, w, G, g, tid, lane, wave, limit;
    int64_t r0;
    uint64_t *slots;
    int *flags;
    int pivots = 0;        // lane j: position chosen for column j
    int first_zero = -1;   // first exactly zero column

    __device__ __forceinline__ static bool stale(uint64_t t, uint32_t seq) {
        return (uint32_t)(t >> 32) != seq;
    }
    __device__ __forceinline__ bool expired(int rounds) {
        if (ll_give_up(rounds, limit, 64, flags)) return true;
        __builtin_amdgcn_s_sleep(1);
        return false;
    }

    // the thread whose row is at position idx writes its columns from CB jb on
    // to d, in the order of its registers (column CB (jb + k) + c at CB k + c)
    __device__ __forceinline__ void put_row(int idx, int jb, T *d) {
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            if (pos[q] == idx) {
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    if (k >= NB - jb) break;   // uniform
#pragma unroll
                    for (int c = 0; c < CB; ++c) d[CB * k + c] = x[q][CB * k + c];
                }
            }
    }

    __device__ __forceinline__ static T lane_value(T t, int l) {   // uniform: lane l's t
        if constexpr (sizeof(T) == 8) {
            const uint64_t b = (uint64_t)__double_as_longlong(t);
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
            return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
        } else {
            return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), l));
        }
    }

    // Column J0 + CB jb + JL of the leaf, J0 the half's first column.
    template <int JL>
    __device__ __forceinline__ void column(WideShared<T, NT, CW> &sh, int J0, int jb) {
        const int JH = CB * jb + JL, J = J0 + JH, par = JL & 1;   // JH: within the half
        const uint32_t seq = (uint32_t)(r0 + J + 1);
        // the wave's candidate: first position >= J of largest |x| (NaN never
        // wins; position J itself stands in when nothing else does)
        int idx, top;
        T piv;
        {
            int h[RPT], hm = -1;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                h[q] = pos[q] >= J ? cand_key(x[q][JL]) : -1;
                hm = max(hm, h[q]);
            }
            top = wave_max_i32(hm);
            uint64_t mask = 0;
            int count = 0;
            T val = x[0][JL];
            int at = pos[0];
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const uint64_t mq = __builtin_amdgcn_ballot_w64(h[q] == top);
                mask |= mq;
                count += __builtin_popcountll(mq);
                if (q > 0) {
                    val = h[q] == top ? x[q][JL] : val;
                    at = h[q] == top ? pos[q] : at;
                }
            }
            int l = __builtin_ctzll(mask);
            bool none = false;
            if (__builtin_expect(top < 0 || count != 1, 0)) {
                if (top < 0) {   // at most one lane of the leaf is at position J
                    mask = 0;
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        mask |= __builtin_amdgcn_ballot_w64(pos[q] == J);
                        val = pos[q] == J ? x[q][JL] : val;
                    }
                    none = mask == 0;
                    l = none ? 0 : __builtin_ctzll(mask);
                    at = J;
                } else {   // ties in the key: by value, then by position
                    double v = -1.0;
                    int i = INT_MAX;
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        const double av = fabs((double)x[q][JL]);
                        if (h[q] == top && (av > v || (av == v && pos[q] < i))) {
                            v = av;
                            i = pos[q];
                            val = x[q][JL];
                        }
                    }
                    at = i;
                    l = first_of(v, i);
                }
            }
            piv = lane_value(val, l);
            idx = none ? INT_MAX : __builtin_amdgcn_readlane(at, l);
            if (NW > 1 && lane == 0) sh.cand[wave] = WideKey{(double)piv, idx, top};
        }
        // the group's candidate: every wave picks it
        int from = 0;
        if constexpr (NW > 1) {
            lds_barrier();
            static_assert(NW == 4 || NW == 8 || NW == 16, "reduced below");
            const WideKey k = sh.cand[lane & (NW - 1)];
            int mx = k.key;
            mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0xB1, 0xF, 0xF, false));
            mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x4E, 0xF, 0xF, false));
            if (NW == 8)
                mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x141, 0xF, 0xF, false));   // row_half_mirror
            if (NW == 16) {
                mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x124, 0xF, 0xF, false));   // row_ror:4
                mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x128, 0xF, 0xF, false));   // row_ror:8
            }
            top = __builtin_amdgcn_readfirstlane(mx);
            uint64_t mask = __builtin_amdgcn_ballot_w64(k.key == top) & (uint64_t)((1 << NW) - 1);
            from = __builtin_ctzll(mask);
            if (__builtin_expect(top < 0 || __builtin_popcountll(mask) != 1, 0)) {
                if (top < 0) {
                    mask = __builtin_amdgcn_ballot_w64(k.idx == J) & (uint64_t)((1 << NW) - 1);
                    from = mask ? __builtin_ctzll(mask) : 0;
                } else {
                    const bool in = lane < NW && k.key == top;
                    from = first_of(in ? fabs(k.v) : -1.0, in ? k.idx : INT_MAX);
                }
            }
            piv = lane_value((T)k.v, from);
            idx = __builtin_amdgcn_readlane(k.idx, from);
        }
        if constexpr (!EXCH) {
            if (wave == from) put_row(idx, jb, sh.row);
        } else {
            uint64_t *gs = slots + (size_t)par * mxlu::kMaxGroups * kSlotWords;
            if (wave == from) {   // the wave that holds the row
                put_row(idx, jb, sh.stage);
                wave_sync_lds();
                const uint32_t *words = reinterpret_cast<const uint32_t *>(sh.stage);
                uint64_t *own = gs + (size_t)g * kSlotWords;
                if (lane < VW * (CW - CB * jb)) ll_store(&own[4 + lane], seq, words[lane]);
                if (lane == 0) ll_store(&own[2], seq, (uint32_t)idx);
            }
            // one batch: the candidates (lane: group) and every NW-th load of
            // rows (GPL groups a load); words not read count as arrived
            const uint64_t none = (uint64_t)seq << 32;
            const bool head = lane < G;
            const uint64_t *ph = gs + (size_t)(head ? lane : 0) * kSlotWords;
            const int rg = GPL * wave + lane / RW;   // group of the first load
            const uint64_t *pr = gs + (size_t)rg * kSlotWords + 4 + lane % RW;
            uint64_t hv0 = none, hv1 = none, hi = none, xw[KR];
            if (head) {
                hv0 = ll_load(ph + 4 + VW * JL);
                if (VW == 2) hv1 = ll_load(ph + 4 + VW * JL + VW - 1);
                hi = ll_load(ph + 2);
            }
#pragma unroll
            for (int k = 0; k < KR; ++k)
                xw[k] = rg + GPL * NW * k < G && lane % RW < VW * (CW - CB * jb)
                            ? ll_load(pr + k * (GPL * NW * kSlotWords))
                            : none;
            for (int rounds = 0;; ++rounds) {
                bool late = stale(hv0, seq) || stale(hv1, seq) || stale(hi, seq);
#pragma unroll
                for (int k = 0; k < KR; ++k) late = late || stale(xw[k], seq);
                if (__builtin_amdgcn_ballot_w64(late) == 0) break;
                if (expired(rounds)) break;
                if (stale(hv0, seq)) hv0 = ll_load(ph + 4 + VW * JL);
                if (VW == 2 && stale(hv1, seq)) hv1 = ll_load(ph + 4 + VW * JL + VW - 1);
                if (stale(hi, seq)) hi = ll_load(ph + 2);
#pragma unroll
                for (int k = 0; k < KR; ++k)
                    if (stale(xw[k], seq)) xw[k] = ll_load(pr + k * (GPL * NW * kSlotWords));
            }
            T hv;
            if constexpr (sizeof(T) == 8)
                hv = __longlong_as_double((long long)(((uint64_t)(uint32_t)hv1 << 32) | (uint32_t)hv0));
            else
                hv = __int_as_float((int)(uint32_t)hv0);
            const int ki = head ? (int)(uint32_t)hi : INT_MAX;
            const int key = ki == INT_MAX ? -1 : cand_key(hv);
            top = wave_max_i32(key);
            uint64_t mask = __builtin_amdgcn_ballot_w64(key == top);
            int gw = __builtin_ctzll(mask);   // the winner's group
            if (__builtin_expect(top < 0 || __builtin_popcountll(mask) != 1, 0)) {
                if (top < 0) {
                    mask = __builtin_amdgcn_ballot_w64(ki == J);
                    gw = mask ? __builtin_ctzll(mask) : 0;
                } else {
                    gw = first_of(key == top ? fabs((double)hv) : -1.0, key == top ? ki : INT_MAX);
                }
            }
            piv = lane_value(hv, gw);
            idx = __builtin_amdgcn_readlane(ki, gw);
            // its row came with one wave's load
            if ((gw / GPL) % NW == wave) {
                uint32_t word = 0;
#pragma unroll
                for (int k = 0; k < KR; ++k)
                    if (gw / (GPL * NW) == k) word = (uint32_t)xw[k];   // uniform
                if (lane / RW == gw % GPL) reinterpret_cast<uint32_t *>(sh.row)[lane % RW] = word;
            }
        }
        // a position outside [J, m) can only follow an expired wait (stale
        // words): position J then, so no index leaves the panel
        int p = idx;
        if (p < J || p >= m) p = J;
        const bool zero = piv == (T)0;
        if (__builtin_expect(zero, 0)) {   // an exactly zero column is left as it is
            p = J;
            if (first_zero < 0) first_zero = J;
        }
        pivots = lane == J ? p : pivots;
        T l[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            pos[q] = pos[q] == p ? J : (pos[q] == J ? p : pos[q]);
            l[q] = zero ? x[q][JL] : x[q][JL] / piv;
            asm("" : "+v"(l[q]));   // here, while the row is on its way
        }
        lds_barrier();   // the row is there
        // One value of the pivot row per lane, in the order of the registers;
        // each goes to the multiply-adds through a scalar register (LDS
        // broadcasts of the whole row to every wave took longer than the
        // arithmetic).
        T ul = sh.row[lane & (CW - 1)];
        asm volatile("" : "+v"(ul));   // read by every lane, not by those of a masked region below
        // Rows up to position J are final: not even a multiple by zero, which
        // an infinity in the pivot row would turn into NaN.
        // The row's values are read by all lanes, outside the masked regions (a
        // region per row and four columns): inside one, what the masked lanes
        // hold would be the register allocator's to choose.  A region per row
        // over all columns with the reads inside took 21 / 30 / 35 / 51 us at 64
        // / 256 / 512 / 1024 rows, now 22 / 31 / 37 / 53, and 102 / 111 at 4096 /
        // 8192, now 91 / 98; with all columns read ahead of it 25 / 32 / 37 / 53
        // and 94 / 102 (scalar registers spill).
        bool below[RPT], some = false;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            below[q] = pos[q] > J;
            some = some || below[q];
            x[q][JL] = below[q] ? l[q] : x[q][JL];
        }
        if (__builtin_amdgcn_ballot_w64(some) == 0) return;   // uniform: no row of the wave's
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (k >= NB - jb) break;   // finished columns (uniform)
            T u[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (CB * k + c > JL) u[c] = lane_value(ul, CB * k + c);
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (below[q]) {
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        if (CB * k + c > JL)
                            x[q][CB * k + c] = fma(-l[q], u[c], x[q][CB * k + c]);
                }
        }
    }

    template <int JL>
    __device__ __forceinline__ void block(WideShared<T, NT, CW> &sh, int J0, int jb) {
        if constexpr (JL < CB) {
            if (J0 + CB * jb + JL < w) {   // uniform
                column<JL>(sh, J0, jb);
                block<JL + 1>(sh, J0, jb);
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
            for (int c = 0; c < CW - CB; ++c) x[q][c] = x[q][c + CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) x[q][CW - CB + c] = t[c];
        }
    }

    // The first half's columns (stored at the rows' positions) taken to the
    // second half's values in x: the pivot rows' unit-lower solve, then every
    // other row's products, one fused multiply-add per term in ascending order
    // as everywhere in the panel.
    __device__ __forceinline__ void second_half(WideShared<T, NT, CW> &sh, const T *P, int64_t lda) {
        if constexpr (!EXCH) {
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (pos[q] >= 0 && pos[q] < CW) {
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        sh.l11[pos[q]][c] = P[(size_t)pos[q] + (size_t)c * lda];
                        sh.u12[pos[q]][c] = x[q][c];
                    }
                }
        } else {
            // the pivot rows lie in several groups: they go through memory,
            // in slots no group uses
            uint64_t *area = slots + (size_t)mxlu::kWideMaxGroups * kSlotWords;
            const uint32_t seq = (uint32_t)(r0 + 1);
            auto put = [&](uint64_t *d, T t) {
                if constexpr (sizeof(T) == 8) {
                    const uint64_t b = (uint64_t)__double_as_longlong(t);
                    ll_store(d, seq, (uint32_t)b);
                    ll_store(d + VW - 1, seq, (uint32_t)(b >> 32));
                } else {
                    ll_store(d, seq, (uint32_t)__float_as_int(t));
                }
            };
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (pos[q] >= 0 && pos[q] < CW) {
                    uint64_t *d = area + pos[q] * RW;
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        put(d + VW * c, P[(size_t)pos[q] + (size_t)c * lda]);
                        put(d + CW * RW + VW * c, x[q][c]);
                    }
                }
            constexpr int kPer = 2 * CW * RW / NT;   // words per thread
            static_assert(2 * CW * RW % NT == 0, "whole words per thread");
            uint64_t word[kPer];
#pragma unroll
            for (int e = 0; e < kPer; ++e) word[e] = ll_load(&area[tid + NT * e]);
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                const int t = tid + NT * e;
                for (int rounds = 0; stale(word[e], seq); ++rounds) {
                    if (expired(rounds)) break;
                    word[e] = ll_load(&area[t]);
                }
                uint32_t *to = reinterpret_cast<uint32_t *>(t < CW * RW ? &sh.l11[0][0] : &sh.u12[0][0]);
                to[t % (CW * RW)] = (uint32_t)word[e];
            }
        }
        __syncthreads();
        if (wave == 0 && lane < CW) {   // a lane per column
            T y[CW];
#pragma unroll
            for (int i = 0; i < CW; ++i) y[i] = sh.u12[i][lane];
#pragma unroll
            for (int k = 0; k < CW; ++k) {
#pragma unroll
                for (int i = k + 1; i < CW; ++i) y[i] = fma(-sh.l11[i][k], y[k], y[i]);
                // (all of l11 in registers would spill: two columns at a time)
                if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < CW; ++i) sh.u12[i][lane] = y[i];
        }
        __syncthreads();
        const T *src[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q) src[q] = P + (pos[q] > 0 ? pos[q] : 0);
#pragma unroll 1
        for (int k0 = 0; k0 < CW; k0 += 8) {
            T lk[8][RPT];
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int q = 0; q < RPT; ++q) lk[k][q] = src[q][(size_t)(k0 + k) * lda];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const T uc = sh.u12[k0 + k][c];
#pragma unroll
                    for (int q = 0; q < RPT; ++q) x[q][c] = fma(-lk[k][q], uc, x[q][c]);
                }
                __builtin_amdgcn_sched_barrier(0);   // (all of u12 in registers would spill)
            }
        }
        // the pivot rows' own values (whatever the products made of them)
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            if (pos[q] >= 0 && pos[q] < CW) {
#pragma unroll
                for (int c = 0; c < CW; ++c) x[q][c] = sh.u12[pos[q]][c];
            }
    }
};

template <typename T, int NT, int RPT, int CW, bool EXCH>
__global__ __launch_bounds__(NT) void panel_leaf_wide_kernel(int m, int w, T *P, int64_t lda, int G,
                                                             int64_t r0, int32_t *__restrict__ ipiv,
                                                             uint64_t *slots, int *flags, int limit) {
    __shared__ WideShared<T, NT, CW> sh;
    using Leaf = WideLeaf<T, NT, RPT, CW, EXCH>;
    Leaf s;
    s.m = m;
    s.w = w;
    s.G = G;
    s.g = blockIdx.x;
    s.tid = threadIdx.x;
    s.lane = s.tid & 63;
    s.wave = __builtin_amdgcn_readfirstlane(s.tid >> 6);
    s.r0 = r0;
    s.slots = slots;
    s.flags = flags;
    s.limit = limit;
    // rows and columns past the leaf: others' values, never looked at (no load
    // is under a condition, so that all are in flight together)
    auto load = [&](int c0) {
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int r = s.g * Leaf::R + s.tid + NT * q;
            const T *src = P + (r < m ? r : m - 1);
#pragma unroll
            for (int c = 0; c < CW; ++c) s.x[q][c] = src[(size_t)min(c0 + c, w - 1) * lda];
        }
    };
    // a row may go to another group's position: every group has loaded these
    // columns of its rows before the exchange (or barrier) of the last of them
    // completed
    auto store = [&](int c0) {
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            if (s.pos[q] >= 0) {
#pragma unroll
                for (int c = 0; c < CW; ++c)
                    if (c0 + c < w) P[(size_t)s.pos[q] + (size_t)(c0 + c) * lda] = s.x[q][c];
            }
    };
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = s.g * Leaf::R + s.tid + NT * q;
        s.pos[q] = r < m ? r : -1;
    }
    for (int J0 = 0; J0 < w; J0 += CW) {   // the halves (or the whole leaf)
        load(J0);
        if (CW < mxlu::kLeafW && J0 > 0) s.second_half(sh, P, lda);
        // With loads still on their way every masked region waits for some, and
        // a region with a wait gets a branch round it: with one row per thread
        // that costs more than the wait for all of them here (the leaves of n =
        // 1024, NB = 64: 1.31 -> 1.28 ms; of more rows 1 to 2 % the other way).
        if (RPT == 1) retire_vector_loads();
        for (int jb = 0; jb < Leaf::NB; ++jb) {
            s.template block<0>(sh, J0, jb);
            s.rotate();   // NB rotations bring the columns back to their registers
        }
        store(J0);
    }
    if (s.g == 0 && s.wave == 0) {
        if (s.lane < w) ipiv[s.lane] = (int32_t)(r0 + s.pivots);
        if (s.lane == 0 && s.first_zero >= 0 && flags[0] == 0) flags[0] = (int)(r0 + s.first_zero + 1);
    }
}

// Interchanges of a leaf (columns [c0, c0 + w) of the kb-column panel at P,
// pivots piv relative to row c0 + base) on the panel's other columns, and those
// of the leaf's second half (from `split` on) on its first half.  A wave per
// column: every wave composes the at most 32 interchanges itself (lane t: row
// t; lane 32 + u: the pivot row of interchange u where it lies below the leaf
// and appears first), then each lane moves one element of a column: all lanes
// have loaded before any stores.
constexpr int kLeafSwapCols = 16;   // columns per workgroup: four per wave

template <typename T>
__global__ __launch_bounds__(256) void panel_leaf_swap_kernel(T *P, int64_t ldp, int64_t m, int kb,
                                                              int c0, int w, int split,
                                                              const int32_t *__restrict__ ipiv,
                                                              int64_t rbase) {
    const int lane = threadIdx.x & 63;
    const int cb = (int)blockIdx.x * kLeafSwapCols + (int)(threadIdx.x >> 6) * 4;
    if (cb >= kb) return;
    // first interchange that applies to these four columns (the leaf and its
    // halves start at multiples of four)
    const int j0 = cb < c0 || cb >= c0 + w ? 0 : (split > 0 && cb < c0 + split ? split : w);
    if (j0 >= w) return;
    // relative pivot rows; one outside [t, m - c0) (possible only after an
    // expired wait) is taken as no interchange
    int pv = lane;
    if (lane < w && lane >= j0) {
        const int64_t q = (int64_t)ipiv[lane] - rbase;
        pv = q >= lane && q < m - c0 ? (int)q : lane;
    }
    int d = lane;
    const int u = lane - 32;
    const int pu = __shfl(pv, u >= 0 ? u : 0);
    if (u >= 0) d = u < w && pu >= w ? pu : -1;
    else if (lane >= w) d = -1;
    int src = d;
#pragma unroll 8
    for (int t = 31; t >= 0; --t) {
        const int q = __builtin_amdgcn_readlane(pv, t);
        if (u > t && q == pu) d = -1;   // the row appeared earlier
        src = src == t ? q : (src == q ? t : src);
    }
    const bool moved = d >= 0 && src != d;
    T v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (moved && cb + e < kb) v[e] = P[(size_t)(c0 + src) + (size_t)(cb + e) * ldp];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (moved && cb + e < kb) P[(size_t)(c0 + d) + (size_t)(cb + e) * ldp] = v[e];
}

}  // namespace

namespace mxlu {

template <typename T>
int panel_leaf_wide(int64_t m, int w, T *P, int64_t ldp, int64_t r0, int32_t *ipiv, int G,
                    const PanelExchange &ex, int *split, hipStream_t s) {
    if (m <= 0 || w <= 0 || w > kLeafW || G > kWideMaxGroups || (int64_t)G * 1024 < m) {
        set_error_msg("panel_leaf_wide: bad shape");
        return MXLU_E_NOMEM;
    }
    *split = 0;
    auto launch = [&](auto kernel, int threads, int groups) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3((unsigned)threads), 0, s, (int)m, w, P, ldp,
                           groups, r0, ipiv + r0, ex.slots, ex.flags, ex.spin_limit);
    };
    // A row per thread as long as one workgroup holds the rows so, then four
    // rows per thread: an exchange through memory costs about 2 us a column, a
    // second wave on every SIMD a quarter, the halves another (2048 rows in
    // one workgroup 72 us, in two 124).  Beyond, two rows per thread with all
    // columns at once (4096 / 8192 / 16384 / 32768 rows 90 / 97 / 116 / 159
    // us) as long as the groups whose rows every wave polls are few, else four
    // rows in halves, whose rows are half as long (106 / 105 / 118 / 145).
    if (m <= 64) launch(panel_leaf_wide_kernel<T, 64, 1, 32, false>, 64, 1);
    else if (m <= 256) launch(panel_leaf_wide_kernel<T, 256, 1, 32, false>, 256, 1);
    else if (m <= 512) launch(panel_leaf_wide_kernel<T, 512, 1, 32, false>, 512, 1);
    else if (m <= 1024) launch(panel_leaf_wide_kernel<T, 1024, 1, 32, false>, 1024, 1);
    else if (m > 2048 && m <= 8192) launch(panel_leaf_wide_kernel<T, 512, 2, 32, true>, 512, G);
    else {
        if (m <= 2048) launch(panel_leaf_wide_kernel<T, 512, 4, 16, false>, 512, 1);
        else launch(panel_leaf_wide_kernel<T, 256, 4, 16, true>, 256, G);
        if (w > 16) *split = 16;   // (the halves)
    }
    MXLU_LAUNCH_CHECK();
    return 0;
}

template <typename T>
int panel_leaf_swap(T *P, int64_t ldp, int64_t m, int64_t kb, int64_t c0, int w, int split,
                    const int32_t *ipiv, int64_t rbase, hipStream_t s) {
    if (kb <= 0 || w <= 0 || w > kLeafW || c0 % 4 || split % 4 || kb > 0x7fffffff - 64) {
        set_error_msg("panel_leaf_swap: bad shape");
        return MXLU_E_NOMEM;
    }
    const unsigned grid = (unsigned)((kb + kLeafSwapCols - 1) / kLeafSwapCols);
    hipLaunchKernelGGL(panel_leaf_swap_kernel<T>, dim3(grid), dim3(256), 0, s, P, ldp, m, (int)kb,
                       (int)c0, w, split, ipiv + rbase, rbase);
    MXLU_LAUNCH_CHECK();
    return 0;
}

}  // namespace mxlu
