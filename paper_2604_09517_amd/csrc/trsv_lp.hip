// Blocked triangular solves in FP32 with the stored 16-bit factor: the
// preconditioner M = U^-1 L^-1 P of the refinement (Sec. II-B).
#include <hip/hip_runtime.h>

#include "common.h"
#include "kernels.h"
#include "lp_common.h"
#include "refine_kernels.h"

namespace {

using namespace mxlu;

// T x = v in one launch, T one of
//   KIND 0: L (unit lower), forward;   KIND 1: U (upper), backward
//   KIND 2: U^T (lower), forward;      KIND 3: L^T (unit upper), backward
// A strip is 64 rows; a wave owns the strip of its place in solve order (lane =
// row), workgroup w the w-th four strips.  It takes the strips before it in
// solve order: those of earlier workgroups as their solutions appear, those of
// its own workgroup through LDS, and solves its own.  Every element takes its
// terms in the order of the textbook substitution (ascending k forward,
// descending k backward), one fused multiply-add each.
//
// What bounds it: the chain of rows (each row waits for the one before) for
// most sizes, and reading the factor, n^2 / 2 values of two bytes, for the
// largest.  So:
//   * a solved row costs the chain a lane read and a multiply-add (L), or the
//     five instructions of the quotient as well (U).  The wave's triangle is
//     in registers as FP32 values, zero from the diagonal on, so that a solved
//     lane keeps its value and no select follows a step.
//   * solutions move on 16 rows at a time: within the workgroup through LDS,
//     to the next one through memory.  The next strip is 16 terms behind when
//     the last row of a strip is solved; the trip from workgroup to workgroup
//     (about 1 us) is paid once in 256 rows.
//   * workgroups further down the chain must keep up with it, and they all
//     stream their rows of the factor meanwhile: each wave keeps four chunks
//     (64 columns of its rows) of 16-byte loads in flight, turns a chunk into
//     rows of consecutive k through registers (column-major factor) and LDS
//     of its own, and asks for the next solutions a block ahead.  No barrier
//     ties the waves of a workgroup until their own strips are next.
// The factor's lanes are 8 x 8 tiles; row r of a staged chunk keeps its eight
// 16-byte units at (unit ^ swz(r)), which spreads rows and units over all
// banks for both the writes and the reads.
//
// A solve with L / U (FP16 or BF16, us): n = 1000: 27 / 34, n = 3001: 77 / 96,
// n = 65536: 1770 / 2080 (reading the factor at 4.3 TB/s takes 1000).  With
// 256-row workgroups that solved their diagonal blocks 64 rows at a time
// between workgroup barriers, staged it in LDS with 2-byte loads and waited
// for a block's solution before asking for the next it was 84 / 148, 250 / 264
// and 2860 / 4590; U^T / L^T at n = 1000: 67 / 75, now 33 / 26.  A block of 256
// rows takes 6.4 us (L) or 8 us (U), about half of it the trip to the next
// workgroup.
//
// Publication: each solved value goes to xs as a 64-bit word holding the
// float's bits and, in the upper half, the launch's tag; writers and readers
// use agent-scope relaxed atomics and a reader polls each word until it
// carries the tag, so no fences are needed.  Tags are unique per launch, so
// words of earlier solves never match.  A workgroup takes its place by an
// atomic ticket when it starts (the counter runs on from launch to launch), so
// that it waits only for workgroups that have started and the chain progresses
// even when not all are resident (by their ids it need not: a workgroup fills a
// CU, and each XCD starts its share of a launch on its own).  The ticket takes
// 2 to 3 us; launches of at most kIdGroups, one on each XCD, go by ids, as it
// would take more of them at once than the device has queues to fill an XCD (the
// gradient of two GMRES solves of n = 1000 takes 3 % longer by tickets).  The
// polling is bounded: on expiry *expired is set and the solve completes with
// invalid values.
constexpr int kStrip = 64;
constexpr int kStrips = kTrsvBs / kStrip;   // strips (waves) of a workgroup
static_assert(kStrips == 4, "one wave per SIMD");

__device__ __forceinline__ uint64_t ll_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float lane_f32(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ int swz(int r) { return ((r >> 1) & 7) ^ ((r >> 4) & 3); }

using Unit = uint32_t __attribute__((ext_vector_type(4)));   // eight 16-bit values

template <int FMT, int KIND>
__global__ __launch_bounds__(256) void trsv_chain_kernel(
    int64_t n, const uint16_t *__restrict__ F, int64_t ldf, const int32_t *__restrict__ perm,
    const double *__restrict__ r, float *__restrict__ v, double *__restrict__ d,
    const unsigned long long *__restrict__ smax, unsigned long long *smax_next, uint64_t *xs,
    uint32_t tag, int nstrips, int *expired, unsigned *ticket, unsigned first_ticket) {
    constexpr bool FWD = KIND == 0 || KIND == 2, UNIT = KIND == 0 || KIND == 3;
    constexpr bool COLS = KIND == 0 || KIND == 1;   // the factor's rows run along its columns
    constexpr bool FIRST = FWD;   // of the two solves
    // a chunk in staging per wave, then the chunks of the own block (those of
    // wave s at s (s + 1) / 2)
    __shared__ Unit stage[kStrips][kStrip][8];
    __shared__ Unit own[kStrips * (kStrips + 1) / 2][kStrip][8];
    __shared__ float xl[kStrips][kStrip];   // solutions of the own block
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int w = (int)blockIdx.x;
    if (gridDim.x > kIdGroups) {
        __shared__ unsigned s_ticket;
        if (threadIdx.x == 0) s_ticket = atomicAdd(ticket, 1u) - first_ticket;
        __syncthreads();
        w = __builtin_amdgcn_readfirstlane((int)s_ticket);
    }
    const int S = kStrips * w + wave;
    const bool active = S < nstrips;
    auto base_of = [&](int s) { return (int64_t)kStrip * (FWD ? s : nstrips - 1 - s); };
    const int64_t r0 = active ? base_of(S) : 0;
    const int64_t row = r0 + lane;
    const bool mine = active && row < n;

    // Chunk of the wave's rows against columns p0 .. p0 + 63
    const int la = lane & 7, lb = lane >> 3;
    auto load = [&](int64_t p0, Unit (&g)[8]) {
        if (r0 + kStrip <= n && p0 + kStrip <= n) {   // uniform
            const uint16_t *src = COLS ? F + (size_t)(r0 + 8 * la) + (size_t)(p0 + 8 * lb) * ldf
                                       : F + (size_t)(p0 + 8 * la) + (size_t)(r0 + lb) * ldf;
            const size_t st = COLS ? (size_t)ldf : 8 * (size_t)ldf;
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = *reinterpret_cast<const Unit *>(src + e * st);
        } else {   // rows and columns past n: others instead, inside the storage
            const int64_t i = COLS ? r0 + 8 * la : p0 + 8 * la;   // first row, column of the first unit
            const int64_t j = COLS ? p0 + 8 * lb : r0 + lb;
            const uint16_t *src = F + (size_t)(i < n ? i : (n - 1) / 8 * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t je = j + (COLS ? e : 8 * e);
                g[e] = *reinterpret_cast<const Unit *>(src + (size_t)(je < n ? je : n - 1) * ldf);
                // columns past n meet a solution of zero, which an infinity
                // would turn into NaN (forward ones never get here)
                if (KIND == 1 && je >= n) g[e] = Unit{0, 0, 0, 0};
            }
            if (KIND == 3) {   // the same (their storage may hold anything)
                Unit keep;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    keep[q] = (i + 2 * q < n ? 0xffffu : 0u) | (i + 2 * q + 1 < n ? 0xffff0000u : 0u);
#pragma unroll
                for (int e = 0; e < 8; ++e) g[e] &= keep;
            }
        }
    };
    auto put = [&](const Unit (&g)[8], Unit (*dst)[8]) {
        if (COLS) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {   // rows 2 q and 2 q + 1 of the tile
                Unit a, b;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    a[m] = __builtin_amdgcn_perm(g[2 * m + 1][q], g[2 * m][q], 0x05040100u);
                    b[m] = __builtin_amdgcn_perm(g[2 * m + 1][q], g[2 * m][q], 0x07060302u);
                }
                const int r = 8 * la + 2 * q;
                dst[r][lb ^ swz(r)] = a;
                dst[r + 1][lb ^ swz(r + 1)] = b;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) dst[lb + 8 * e][la ^ swz(lb + 8 * e)] = g[e];
        }
    };
    // the lane's row of a staged chunk: word p holds columns 2 p and 2 p + 1
    auto get = [&](Unit (*src)[8], uint32_t (&rr)[32]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const Unit u = src[lane][j ^ swz(lane)];
#pragma unroll
            for (int m = 0; m < 4; ++m) rr[4 * j + m] = u[m];
        }
    };
    auto value = [&](const uint32_t (&rr)[32], int k) {
        const uint32_t u = rr[k >> 1];
        if (FMT == kFmtBf16) return __uint_as_float((k & 1) ? u & 0xffff0000u : u << 16);
        return lp_to_f32<FMT>((uint16_t)((k & 1) ? u >> 16 : u));
    };
    // the right-hand side: r / s in FP32 (P r / s for L), or the first solution
    const double scale = __longlong_as_double((long long)*smax);
    float acc = 0.0f;
    if (FIRST) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *smax_next = 0;
        if (mine) {
            const double ri = r[KIND == 0 && perm ? perm[row] : row];
            acc = scale > 0.0 ? (float)(ri / scale) : 0.0f;
        }
    } else if (mine) {
        acc = v[row];
    }
    // terms of 16 columns (group gq of the chunk in solve order), x: lane = column
    auto terms = [&](const uint32_t (&rr)[32], float x, auto gq) {
        constexpr int g = decltype(gq)::value;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int k = FWD ? 16 * g + e : 63 - 16 * g - e;
            acc = fmaf(-value(rr, k), lane_f32(x, k), acc);
        }
    };
    using G0 = std::integral_constant<int, 0>;
    using G1 = std::integral_constant<int, 1>;
    using G2 = std::integral_constant<int, 2>;
    using G3 = std::integral_constant<int, 3>;
    // solution words of strip s, a word per lane; columns past n as arrived zeros
    auto ask = [&](int s) {
        const int64_t c = base_of(s) + lane;
        return c < n ? ll_load(&xs[c]) : (uint64_t)tag << 32;
    };
    auto there = [&](uint64_t x) { return (uint32_t)(x >> 32) == tag; };
    // a wait gives up after long polling, or when another one has
    auto expire = [&](int spins) {
        if ((spins & 0xfff) != 0xfff) return false;
        if (spins >= (1 << 24)) atomicExch(expired, 1);   // about 10 s
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(expired, __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT)) != 0;
    };

    // the own block's chunks; of the last, the own strip's, only the triangle
    // is kept: zero from the diagonal on and in rows past n
    Unit(*diag)[8] = own[wave * (wave + 1) / 2 + wave];
    uint32_t rr[32];
    if (active) {
        Unit g[kStrips][8];
#pragma unroll
        for (int s = 0; s < kStrips; ++s)
            if (s <= wave) load(base_of(kStrips * w + s), g[s]);
#pragma unroll
        for (int s = 0; s < kStrips; ++s)
            if (s <= wave) put(g[s], own[wave * (wave + 1) / 2 + s]);
        wave_sync_lds();
        get(diag, rr);
        wave_sync_lds();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            Unit u;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int k = 8 * j + 2 * m;
                const uint32_t keep = ((FWD ? k < lane : k > lane) ? 0xffffu : 0u) |
                                      ((FWD ? k + 1 < lane : k + 1 > lane) ? 0xffff0000u : 0u);
                u[m] = mine ? rr[4 * j + m] & keep : 0u;
            }
            diag[lane][j ^ swz(lane)] = u;
        }
        wave_sync_lds();
    }
    uint32_t tri[32];   // read ahead of the chain
    get(diag, tri);
#pragma unroll
    for (int p = 0; p < 32; ++p) asm volatile("" : "+v"(tri[p]));
    float dl = 1.0f;   // the row's diagonal entry
    if (!UNIT && mine) dl = lp_to_f32<FMT>(F[(size_t)row + (size_t)row * ldf]);
    const float rdiag = UNIT ? 1.0f : 1.0f / dl;

    if (w > 0 && active) {
        Unit ring[kStrips][8];   // the next block's chunks
        uint64_t xw[kStrips];    // and its solution words
#pragma unroll
        for (int c = 0; c < kStrips; ++c) load(base_of(c), ring[c]);
        if (w > 1)
#pragma unroll
            for (int c = 0; c < kStrips; ++c) xw[c] = ask(c);
        for (int b = 0; b + 1 < w; ++b) {
            bool late = false;
#pragma unroll
            for (int c = 0; c < kStrips; ++c) late = late || !there(xw[c]);
            if (__builtin_amdgcn_ballot_w64(late)) {
                // one lane watches the word that appears last, with pauses as
                // long as the block is far ahead of the own one: pollers
                // crowd the producer's stores
                if (lane == 0) {
                    const int64_t pb = base_of(kStrips * b + kStrips - 1);
                    const uint64_t *p = &xs[FWD ? (pb + kStrip <= n ? pb + kStrip - 1 : n - 1) : pb];
                    for (int spins = 0; !there(ll_load(p)) && !expire(spins); ++spins)
                        for (int q = 0; q < w - b && q < 16; ++q) __builtin_amdgcn_s_sleep(8);
                }
                for (int spins = 0;; ++spins) {
                    late = false;
#pragma unroll
                    for (int c = 0; c < kStrips; ++c) {
                        xw[c] = ask(kStrips * b + c);
                        late = late || !there(xw[c]);
                    }
                    if (__builtin_amdgcn_ballot_w64(late) == 0 || expire(spins)) break;
                }
            }
            float x[kStrips];
#pragma unroll
            for (int c = 0; c < kStrips; ++c) x[c] = __uint_as_float((uint32_t)xw[c]);
            if (b + 2 < w)
#pragma unroll
                for (int c = 0; c < kStrips; ++c) xw[c] = ask(kStrips * (b + 1) + c);
#pragma unroll
            for (int c = 0; c < kStrips; ++c) {
                put(ring[c], stage[wave]);
                load(base_of(kStrips * (b + 1) + c), ring[c]);
                wave_sync_lds();
                get(stage[wave], rr);
                wave_sync_lds();
                terms(rr, x[c], G0{});
                terms(rr, x[c], G1{});
                terms(rr, x[c], G2{});
                terms(rr, x[c], G3{});
            }
        }
        // the last earlier block is on the chain: 16 columns at a time as
        // they appear
#pragma unroll
        for (int c = 0; c < kStrips; ++c) {
            put(ring[c], stage[wave]);
            wave_sync_lds();
            get(stage[wave], rr);
            wave_sync_lds();
            uint64_t x = 0, ok = 0;
            auto group = [&](auto gq) {
                constexpr int g = decltype(gq)::value;
                constexpr uint64_t mask = 0xffffull << (16 * (FWD ? g : 3 - g));
                for (int spins = 0; (ok & mask) != mask; ++spins) {
                    // the later waves are not next: fewer polls for them
                    if (wave > 0) __builtin_amdgcn_s_sleep(6);
                    if (!there(x)) x = ask(kStrips * (w - 1) + c);
                    ok = __builtin_amdgcn_ballot_w64(there(x));
                    if (expire(spins)) break;
                }
                terms(rr, __uint_as_float((uint32_t)x), gq);
            };
            group(G0{});
            group(G1{});
            group(G2{});
            group(G3{});
        }
    }
    // own block, strip by strip
    for (int s = 0; s < kStrips; ++s) {
        if (wave > s) {
            // strip s's solution, 16 rows behind its solver
            if (active) get(own[wave * (wave + 1) / 2 + s], rr);
            auto group = [&](auto gq) {
                lds_barrier();
                const float x = xl[s][lane];
                if (active) terms(rr, x, gq);
            };
            group(G0{});
            group(G1{});
            group(G2{});
            group(G3{});
        } else if (wave == s && active) {
            float x = mine ? acc : 0.0f, sol = 0.0f;
            // U: the quotient x / d of a step comes from r = RN(1/d), formed
            // ahead of the chain: q0 = RN(x r), q = RN(q0 + (x - q0 d) r) with
            // both corrections fused multiply-adds.  While every value stays
            // in the normal range that is the correctly rounded quotient
            // (Markstein's theorem for a reciprocal rounded to nearest; also
            // checked against the division on 4e8 operand pairs, quotients at
            // rounding midpoints and divisors with all-ones significands
            // included, and scale-invariant away from underflow and overflow).
            // After each 16 steps one vote checks |x| >= 2^-100 (or x == 0),
            // |q| within [2^-99, 2^99] and |d| within [2^-100, 2^100] of the
            // lanes solved, and if any is outside (or, for L, not finite: the
            // zeros of the triangle would turn it into NaN in solved lanes),
            // the steps are taken again with the division and a select: the
            // result is the division's bit for bit either way.
            auto quotient = [&](float y) {
                if (UNIT) return y;
                const float q0 = y * rdiag;
                return fmaf(fmaf(-q0, dl, y), rdiag, q0);
            };
            auto group = [&](auto gq) {
                constexpr int g = decltype(gq)::value;
                const float x_in = x;
                constexpr uint64_t lanes = 0xffffull << (16 * (FWD ? g : 3 - g));
                const bool here = (FWD ? lane >> 4 : 3 - (lane >> 4)) == g;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int k = FWD ? 16 * g + e : 63 - 16 * g - e;
                    x = fmaf(-value(tri, k), lane_f32(quotient(x), k), x);
                }
                const float q = quotient(x);
                const float ax = fabsf(x), aq = fabsf(q), ad = fabsf(dl);
                const bool in = UNIT ? aq <= 0x1.fffffep127f
                                     : (x == 0.0f || (ax >= 0x1p-100f && aq >= 0x1p-99f && aq <= 0x1p99f)) &&
                                           ad >= 0x1p-100f && ad <= 0x1p100f;
                sol = here ? q : sol;
                if (__builtin_expect((__builtin_amdgcn_ballot_w64(in) & lanes) != lanes, 0)) {
                    x = x_in;
#pragma unroll 1
                    for (int e = 0; e < 16; ++e) {
                        const int k = FWD ? 16 * g + e : 63 - 16 * g - e;
                        const float xk = lane_f32(UNIT ? x : x / dl, k);
                        const Unit u = diag[lane][(k >> 3) ^ swz(lane)];
                        const uint32_t h = u[(k >> 1) & 3];
                        const float f = lp_to_f32<FMT>((uint16_t)((k & 1) ? h >> 16 : h));
                        sol = lane == k ? xk : sol;
                        if ((FWD ? k < lane : k > lane) && mine) x = fmaf(-f, xk, x);
                    }
                }
                xl[s][lane] = sol;   // (lanes not solved yet write again)
                if (here && mine)
                    __hip_atomic_store(&xs[row], ((uint64_t)tag << 32) | __float_as_uint(sol),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                lds_barrier();
            };
            group(G0{});
            group(G1{});
            group(G2{});
            group(G3{});
            if (FIRST) {
                if (mine) v[row] = sol;
            } else if (mine) {   // d = s x (P^T of it for L^T)
                d[KIND == 3 && perm ? perm[row] : row] = scale > 0.0 ? scale * (double)sol : 0.0;
            }
        } else {
            for (int g = 0; g < 4; ++g) lds_barrier();
        }
    }
}

template <int FMT, int KIND>
int trsv_run(int64_t n, const uint16_t *F, int64_t ldf, const int32_t *perm, const double *r, double *d,
             float *v, const unsigned long long *smax, unsigned long long *smax_next, TrsvChain &ch,
             hipStream_t s) {
    const int64_t nstrips = (n + kStrip - 1) / kStrip;
    if (nstrips > 0x7ffffff0) {
        set_error_msg("trsv: too many blocks");
        return MXLU_E_NOMEM;
    }
    if (((uintptr_t)F % 16) || (ldf % 8)) {
        set_error_msg("trsv: factor storage must be 16-byte aligned with ldf % 8 == 0");
        return MXLU_E_NOMEM;
    }
    const uint32_t tag = ++ch.tag;
    const unsigned groups = (unsigned)((nstrips + kStrips - 1) / kStrips);
    hipLaunchKernelGGL((trsv_chain_kernel<FMT, KIND>), dim3(groups), dim3(256), 0, s, n, F, ldf, perm, r,
                       v, d, smax, smax_next, ch.xs, tag, (int)nstrips, ch.expired, ch.ticket,
                       ch.tickets);
    MXLU_LAUNCH_CHECK();
    if (groups > kIdGroups) ch.tickets += groups;   // (modulo 2^32, as the counter)
    return 0;
}

template <int FMT>
int apply(int trans, int64_t n, const uint16_t *F, int64_t ldf, const int32_t *perm, const double *r,
          double *d, float *v, const unsigned long long *smax, unsigned long long *smax_next,
          TrsvChain &ch, hipStream_t s) {
    if (trans) {   // v = r / s; U^T; L^T; P^T
        MXLU_TRY((trsv_run<FMT, 2>(n, F, ldf, perm, r, d, v, smax, smax_next, ch, s)));
        return trsv_run<FMT, 3>(n, F, ldf, perm, r, d, v, smax, smax_next, ch, s);
    }
    // v = P r / s; L; U
    MXLU_TRY((trsv_run<FMT, 0>(n, F, ldf, perm, r, d, v, smax, smax_next, ch, s)));
    return trsv_run<FMT, 1>(n, F, ldf, perm, r, d, v, smax, smax_next, ch, s);
}

}  // namespace

namespace mxlu {

int lp_precond_apply(int fmt, int trans, int64_t n, const uint16_t *F, int64_t ldf,
                     const int32_t *perm, const double *r, double *d, float *v32,
                     const unsigned long long *smax, unsigned long long *smax_next, TrsvChain &ch,
                     hipStream_t s) {
    if (n <= 0) return 0;
    return fmt == kFmtBf16
               ? apply<kFmtBf16>(trans, n, F, ldf, perm, r, d, v32, smax, smax_next, ch, s)
               : apply<kFmtFp16>(trans, n, F, ldf, perm, r, d, v32, smax, smax_next, ch, s);
}

}  // namespace mxlu
