// Triangular solves with the FP64 factors (the solve phase of Sec. III-A.1 and
// its transpose) for up to 16 right-hand sides at a time, and the row
// permutation that the interchanges amount to.
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "quarter.h"

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// T X = B for up to 16 right-hand sides in one launch, T one of
//   KIND 0: L (unit lower), forward      KIND 1: U (upper), backward
//   KIND 2: U^T (lower), forward         KIND 3: L^T (unit upper), backward
// Workgroup w owns the w-th block of kTriRows rows in solve order; wave v of
// it owns 16 of those rows, with all right-hand sides as one 16 x 16 FP64
// matrix-core accumulator.  It applies the solutions of the earlier blocks as
// they appear (their factor entries are loaded one block ahead), then solves
// its own block 16 rows at a time: the owning wave by substitution, four rows
// a step, the later waves apply the result with the matrix cores.
//
// What bounds it is the chain of blocks, not the n^2 / 2 factor entries: per
// block one trip of the solution from workgroup to workgroup and eight
// dependent 16-row solves.  Blocks of 128 rows share that trip among more
// rows than smaller ones and still leave n / 128 compute units streaming the
// factor.  Before, every 256 rows took two launches (a diagonal block on one
// workgroup with a barrier per row, and a row-per-thread update):
// n = 8192, 16 right-hand sides: 18.0 -> 1.13 ms; n = 32768, one: 12.4 -> 4.4
// (measured with the factors of a matrix of the benchmark recipe).
// A block takes 7.5 us (L) and 8.6 us (U): eight strips of about 0.7 us and 2
// us for the way to the next workgroup.  With the accumulators' rows spread over
// the quarter waves the other way, each step exchanged its four rows among all
// quarters first, and a block took 8.6 and 9.3 us; a substitution with a lane
// per right-hand side (16 values in registers, factor entries broadcast from
// LDS) waited for an LDS read every other multiply-add and took 2.5 times as
// long.
//
// A solution value goes to `out` as one 64-bit word, written and read with
// agent-scope relaxed atomics; the words start as kTriEmpty, a signalling NaN
// that no arithmetic produces, and a reader polls a word until it holds
// anything else, so no flags and fences are needed.  A workgroup takes its
// block by an atomic ticket when it starts, so that it waits only for
// workgroups that have started and the chain advances however many are
// resident: a workgroup fills a CU, each XCD starts its share of a launch on its
// own, and going by their ids two solves on two streams could each fill an XCD
// and wait for a block of the other's.  The ticket takes 2 to 3 us of a launch;
// launches of at most kIdGroups workgroups, one on each XCD, go by their ids: to
// fill an XCD takes more of them at once than the device has queues.
// The polling is bounded: a wait that expires goes on with NaN, sets *expired,
// which ends the launch's other waits, and is counted (mxlu_solve_timeouts).
// ---------------------------------------------------------------------------
constexpr int kTriRows = 128;
constexpr int kTriLd = 17;   // LDS row of 16 right-hand sides (odd: columns spread over the banks)
constexpr uint64_t kTriEmpty = 0x7FF000005EED0001ull, kTriNaN = 0x7FF8000000000000ull;

// launches whose waits have expired since the process started
__device__ unsigned g_tri_timeouts;

__global__ __launch_bounds__(256) void tri_clear_kernel(int64_t n, int nr, double *__restrict__ X,
                                                        int64_t ldx, mxlu::TriSync *__restrict__ sync) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0) sync->ticket = sync->expired = 0;
    if (i >= n) return;
    for (int c = 0; c < nr; ++c)
        X[(size_t)i + (size_t)c * (size_t)ldx] = __longlong_as_double((long long)kTriEmpty);
}

__device__ __forceinline__ uint64_t tri_load(const double *p) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

template <int KIND>
__global__ __launch_bounds__(512) void tri_chain_f64_kernel(
    int64_t n, int nr, const double *__restrict__ T, int64_t ldt, const double *in, int64_t ldin,
    const int32_t *__restrict__ inperm, double *out, int64_t ldo,
    const int32_t *__restrict__ outperm, int nblk, mxlu::TriSync *sync, int max_spins) {
    constexpr bool TR = KIND >= 2, FWD = KIND == 0 || KIND == 2, UNIT = KIND == 0 || KIND == 3;
    constexpr int BS = kTriRows, NS = BS / 16;
    __shared__ double Xs[2][BS][kTriLd];
    // tiles of -F of the own block between different strips, in operand order
    __shared__ double Ot[NS * (NS - 1) / 2][4][64];
    __shared__ __attribute__((aligned(16))) double Dg[NS][16][16];   // Dg[s][k][i] = F[16s+i][16s+k]
    __shared__ double Rd[BS];           // reciprocals of the diagonal
    __shared__ int s_range[NS];         // the strip's diagonal is in the normal range
    __shared__ unsigned s_ticket;
    const int tid = threadIdx.x, lane = tid & 63;
    const int v = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;
    int w = blockIdx.x;
    if (nblk > mxlu::kIdGroups) {
        if (tid == 0) s_ticket = atomicAdd(&sync->ticket, 1u);
        __syncthreads();
        w = __builtin_amdgcn_readfirstlane((int)s_ticket);
    }
    const int64_t r0 = (int64_t)(FWD ? w : nblk - 1 - w) * BS;
    // this lane's factor row: matrix row i stands for row 4 (i % 4) + i / 4 of
    // the strip, so that a quarter wave's accumulators are four rows in turn
    const int ri = 4 * (li & 3) + (li >> 2);
    const int64_t row = r0 + 16 * v + ri;
    const int64_t rowc = row < n ? row : n - 1;
    auto block_row = [&](int t) { return (int64_t)(FWD ? t : nblk - 1 - t) * BS; };
    auto tile = [&](int vv, int s) {   // of strip vv's rows and strip s's columns, s solved before vv
        const int i = FWD ? vv : NS - 1 - vv, j = FWD ? s : NS - 1 - s;
        return i * (i - 1) / 2 + j;
    };

    // -F of the wave's 16 rows, columns p0 .. p0 + BS: lane (li, lq), entry kk
    // is -F[row][p0 + 4 kk + lq] (F: the effective lower or upper factor);
    // rows and columns past n are zero.  L and L^T: F itself, the earlier blocks'
    // solutions are negated instead, so that nothing waits for the loads before
    // their block's turn (L, n = 2047 / 12001: 165 / 980 -> 139 / 855 us; U^T
    // takes 172 for 151 that way, U the same).
    constexpr bool NEGX = UNIT;
    auto load_f = [&](int64_t p0, double (&a)[BS / 4]) {
        if (p0 + BS <= n && r0 + 16 * v + 16 <= n) {   // uniform
            const double *src = TR ? T + (size_t)(p0 + lq) + (size_t)row * (size_t)ldt
                                   : T + (size_t)row + (size_t)(p0 + lq) * (size_t)ldt;
            const size_t st = TR ? 4 : 4 * (size_t)ldt;
#pragma unroll
            for (int kk = 0; kk < BS / 4; ++kk) a[kk] = NEGX ? src[kk * st] : -src[kk * st];
        } else {
#pragma unroll
            for (int kk = 0; kk < BS / 4; ++kk) {
                const int64_t k = p0 + 4 * kk + lq, kc = k < n ? k : n - 1;
                const double f = TR ? T[(size_t)kc + (size_t)rowc * (size_t)ldt]
                                    : T[(size_t)rowc + (size_t)kc * (size_t)ldt];
                a[kk] = row < n && k < n ? (NEGX ? f : -f) : 0.0;
            }
        }
    };
    auto word = [&](int64_t g, int c) -> const double * {
        return out + (size_t)(outperm ? outperm[g] : g) + (size_t)c * (size_t)ldo;
    };
    // solution words of the block at p0: thread (row tid % BS, right-hand
    // sides tid / BS + 4 e); rows and columns that do not exist are zero
    const int xr = tid & (BS - 1), xc = tid / BS;
    auto operand = [](uint64_t x) {   // of the products with F as loaded
        const double d = __longlong_as_double((long long)x);
        return NEGX ? -d : d;
    };
    uint64_t xw[4];
    auto load_x = [&](int64_t p0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            xw[e] = (p0 + xr < n && xc + 4 * e < nr) ? tri_load(word(p0 + xr, xc + 4 * e)) : 0ull;
    };
    // a wait gives up after max_spins looks (2^24: 16 s or more), or when another
    // one has
    auto give_up = [&](int spins) {
        if (spins >= max_spins) {
            if (atomicExch(&sync->expired, 1u) == 0) atomicAdd(&g_tri_timeouts, 1u);
            return true;
        }
        return (spins & 1023) == 1023 && __hip_atomic_load(&sync->expired, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT) != 0;
    };
    // wait for them: one lane of the workgroup watches the word that appears
    // last, with long pauses, so that the many workgroups further down the
    // chain do not crowd the producer's stores; then every thread reads its
    // own (looking again at the few that are not there yet)
    auto await_x = [&](int64_t p0) {
        if (tid == 0) {
            const int64_t last = FWD ? (p0 + BS < n ? p0 + BS - 1 : n - 1) : p0;
            const double *p = word(last, nr - 1);
            for (int k = 0; tri_load(p) == kTriEmpty && !give_up(k); ++k)
                __builtin_amdgcn_s_sleep(16);
        }
        __syncthreads();
        load_x(p0);
        for (int rounds = 0;; ++rounds) {
            bool late = false;
#pragma unroll
            for (int e = 0; e < 4; ++e) late = late || xw[e] == kTriEmpty;
            if (__builtin_amdgcn_ballot_w64(late) == 0) return;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (xw[e] == kTriEmpty)
                    xw[e] = give_up(rounds) ? kTriNaN : tri_load(word(p0 + xr, xc + 4 * e));
        }
    };

    double a[BS / 4], an[BS / 4];
    // the own block: off-diagonal tiles and the diagonal tile of each strip
    // (rows past n as the identity) wait in LDS
    load_f(r0, a);
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (FWD ? s < v : s > v) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) Ot[tile(v, s)][kk][lane] = NEGX ? -a[4 * s + kk] : a[4 * s + kk];
        }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int64_t k = r0 + 16 * v + 4 * kk + lq, kc = k < n ? k : n - 1;
        const double f = TR ? T[(size_t)kc + (size_t)rowc * (size_t)ldt]
                            : T[(size_t)rowc + (size_t)kc * (size_t)ldt];
        Dg[v][4 * kk + lq][ri] = row < n && k < n ? f : (row == k ? 1.0 : 0.0);
    }
    if (!UNIT) {
        wave_sync_lds();
        const double d = Dg[v][li][li];
        if (lq == 0) Rd[16 * v + li] = 1.0 / d;
        const bool in_range = fabs(d) >= 0x1p-500 && fabs(d) <= 0x1p500;
        const uint64_t all = __builtin_amdgcn_ballot_w64(in_range);
        if (lane == 0) s_range[v] = all == ~0ull;
    }
    v4d acc;                   // lane (li, lq), register r: row 4 lq + r, right-hand side li
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t g = r0 + 16 * v + 4 * lq + r;
        acc[r] = (g < n && li < nr) ? in[(size_t)(inperm ? inperm[g] : g) + (size_t)li * (size_t)ldin]
                                    : 0.0;
    }
    if (w > 0) load_f(block_row(0), a);
    for (int t = 0; t + 1 < w; ++t) {
        await_x(block_row(t));
        double(*X)[kTriLd] = Xs[t & 1];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            X[xr][xc + 4 * e] = operand(xw[e]);
        lds_barrier();
        load_f(block_row(t + 1), an);
        // a block's products are summed by themselves: n / 128 partial sums
        // round less than one running sum of n terms
        v4d sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < BS / 4; ++kk)
            sum = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kk], X[4 * kk + lq][li], sum, 0, 0, 0);
        acc += sum;
#pragma unroll
        for (int kk = 0; kk < BS / 4; ++kk) a[kk] = an[kk];
    }
    // The strip's diagonal tile for the substitution, in solve order: step b
    // takes rows o(4 b) .. o(4 b + 3).  tri: its 4 x 4 triangle (uniform),
    // ta: the tile's rows still to come against the step's four columns, as a
    // matrix-core operand (zero for rows already solved).
    auto ord = [](int e) { return FWD ? e : 15 - e; };   // row or column of solve order e
    double tri[4][6], ta[4], dv[4][4], rv[4][4];
    wave_sync_lds();   // Dg[v], Rd: this wave's own
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int i = 1, e = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < i; ++k, ++e) tri[b][e] = Dg[v][ord(4 * b + k)][ord(4 * b + i)];
        if (!UNIT) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dv[b][i] = Dg[v][ord(4 * b + i)][ord(4 * b + i)];
                rv[b][i] = Rd[16 * v + ord(4 * b + i)];
            }
        }
        const int g = FWD ? b : 3 - b;   // rows and columns 4 g .. 4 g + 3
        ta[b] = (FWD ? ri > 4 * g + 3 : ri < 4 * g) ? -Dg[v][4 * g + lq][ri] : 0.0;
    }
    if (w > 0) {
        // the last earlier block is on the chain's critical path: its strips
        // are taken one by one as they appear, so that after the last of them
        // only four matrix instructions per wave remain
        const int64_t p0 = block_row(w - 1);
        double(*X)[kTriLd] = Xs[(w - 1) & 1];
        const int sr = tid & 15, sc = (tid >> 4) & 15;
        v4d sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int s = FWD ? j : NS - 1 - j;
            if (tid < 256) {
                const int64_t g = p0 + 16 * s + sr;
                uint64_t x = 0;
                if (g < n && sc < nr) {
                    const double *p = word(g, sc);
                    x = tri_load(p);
                    for (int spins = 0; x == kTriEmpty; ++spins) {
                        __builtin_amdgcn_s_sleep(1);
                        x = give_up(spins) ? kTriNaN : tri_load(p);
                    }
                }
                X[16 * s + sr][sc] = operand(x);
            }
            lds_barrier();
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                sum = __builtin_amdgcn_mfma_f64_16x16x4f64(a[4 * s + kk], X[16 * s + 4 * kk + lq][li],
                                                           sum, 0, 0, 0);
        }
        acc += sum;
    }
    // own block, 16 rows at a time
    double(*X)[kTriLd] = Xs[w & 1];
    lds_barrier();   // Ot is complete; Xs[w & 1] was last read two blocks ago
    // Substitution with the wave's tile, four rows a step: quarter wave g holds
    // rows 4 g .. 4 g + 3 of its lanes' right-hand sides, which each lane solves
    // by itself; three lane permutes of a word turn them into a matrix operand
    // (lane (li, lq): row 4 g + lq), and one matrix instruction takes them to
    // the rows still to come.  x[g]: that operand, the solution.
    // U: the quotient x / d through r = RN(1 / d), formed ahead of the chain:
    // q0 = RN(x r), q = RN(q0 + (x - q0 d) r), the correctly rounded quotient
    // while everything, x - q0 d (down to 2^-105 x) included, stays in the normal
    // range (Markstein's theorem); DIV divides.  Returned: whether it did, for d
    // within [2^-500, 2^500]: quotients up to 2^900, and numerators of 2^-390 at
    // least or zero (whose exponent reads as 0; looking at the numerators takes U's
    // chain of n = 8192, 16 right-hand sides from 526 to 548 us).
    auto substitute = [&](auto div, double (&x)[4]) -> bool {
        constexpr bool DIV = decltype(div)::value;
        v4d c = acc;
        uint32_t top = 0;
        int low = 0;
        auto step = [&](auto bq) {
            constexpr int b = decltype(bq)::value, g = FWD ? b : 3 - b;
            double y[4];   // in solve order
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = c[FWD ? i : 3 - i];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!UNIT) {
                    if (DIV) {
                        y[i] = y[i] / dv[b][i];
                    } else {
                        low = min(low, __builtin_amdgcn_frexp_exp(y[i]));
                        const double q0 = y[i] * rv[b][i];
                        y[i] = fma(fma(-q0, dv[b][i], y[i]), rv[b][i], q0);
                    }
                }
#pragma unroll
                for (int k = i + 1; k < 4; ++k)
                    y[k] = fma(-tri[b][k * (k - 1) / 2 + i], y[i], y[k]);
            }
            const double z[4] = {y[FWD ? 0 : 3], y[FWD ? 1 : 2], y[FWD ? 2 : 1], y[FWD ? 3 : 0]};
            x[g] = spread<g>(z);
            if (!UNIT && !DIV)
                top = max(top, (uint32_t)((uint64_t)__double_as_longlong(x[g]) >> 32) & 0x7fffffffu);
            if (b < 3) c = __builtin_amdgcn_mfma_f64_16x16x4f64(ta[b], x[g], c, 0, 0, 0);
        };
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
        return top < 0x78300000u && low >= -389;
    };
    for (int j = 0; j < NS; ++j) {
        const int s = FWD ? j : NS - 1 - j;
        if (v == s) {
            double x[4];
            const bool in = substitute(std::false_type{}, x);
            if (!UNIT && (!__all(in) || !s_range[s])) substitute(std::true_type{}, x);   // wave-uniform
#pragma unroll
            for (int r = 0; r < 4; ++r) X[16 * s + lq + 4 * r][li] = x[r];
        }
        lds_barrier();
        if (FWD ? v > s : v < s) {   // wave-uniform: later strips take strip s's solution
            const double(*O)[64] = Ot[tile(v, s)];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(O[kk][lane], X[16 * s + 4 * kk + lq][li], acc,
                                                           0, 0, 0);
        } else if (v == s) {
            // publish: 16 rows of one right-hand side per quarter wave
            uint64_t b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                b[e] = (uint64_t)__double_as_longlong(X[16 * s + li][lq + 4 * e]);
                if (b[e] == kTriEmpty) b[e] |= 0x0008000000000000ull;   // a quiet NaN then
            }
            const int64_t g = r0 + 16 * s + li;
            if (g < n) {
                double *o = out + (size_t)(outperm ? outperm[g] : g);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (lq + 4 * e < nr)
                        __hip_atomic_store(
                            reinterpret_cast<uint64_t *>(o + (size_t)(lq + 4 * e) * (size_t)ldo), b[e],
                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

template <int KIND>
int tri_chain(int64_t n, int nr, const double *T, int64_t ldt, const double *in, int64_t ldin,
              const int32_t *inperm, double *out, int64_t ldo, const int32_t *outperm,
              mxlu::TriSync *sync, hipStream_t s) {
    const int64_t nblk = (n + kTriRows - 1) / kTriRows;
    hipLaunchKernelGGL(tri_clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, nr,
                       out, ldo, sync);
    MXLU_LAUNCH_CHECK();
    hipLaunchKernelGGL(tri_chain_f64_kernel<KIND>, dim3((unsigned)nblk), dim3(512), 0, s, n, nr, T,
                       ldt, in, ldin, inperm, out, ldo, outperm, (int)nblk, sync,
                       mxlu::g_expire_waits.load() ? 0 : 1 << 24);
    MXLU_LAUNCH_CHECK();
    return 0;
}

}  // namespace

namespace mxlu {

int tri_solve_f64(int64_t n, int nr, const double *LU, int64_t lda, const int32_t *perm, double *B,
                  int64_t ldb, int trans, double *E, int64_t lde, TriSync *sync, hipStream_t s) {
    if (n <= 0 || nr <= 0) return 0;
    if (nr > 16) {
        set_error_msg("tri_solve_f64: more than 16 right-hand sides");
        return MXLU_E_NOMEM;
    }
    if (trans == 0) {   // L y = P b, U x = y
        MXLU_TRY(tri_chain<0>(n, nr, LU, lda, B, ldb, perm, E, lde, nullptr, sync, s));
        return tri_chain<1>(n, nr, LU, lda, E, lde, nullptr, B, ldb, nullptr, sync, s);
    }
    // U^T y = b, L^T z = y, x = P^T z
    MXLU_TRY(tri_chain<2>(n, nr, LU, lda, B, ldb, nullptr, E, lde, nullptr, sync, s));
    return tri_chain<3>(n, nr, LU, lda, E, lde, nullptr, B, ldb, perm, sync, s);
}

int tri_timeouts(int64_t *count) {
    unsigned c = 0;
    MXLU_HIP_TRY(hipMemcpyFromSymbol(&c, HIP_SYMBOL(g_tri_timeouts), sizeof(c)));
    *count = c;
    return 0;
}

}  // namespace mxlu
