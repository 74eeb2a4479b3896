// SWAP of the right-looking LU (Sec. III-A.1): a step's row interchanges on
// the columns right of its panel, and the deferred ones left of the panels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "common.h"
#include "kernels.h"

namespace {

// ---------------------------------------------------------------------------
// The row whose content interchanges u = 0 .. end up in row d is found by
// taking them in reverse: src <- q_u where src == u, src <- u where src == q_u.
// As q_u >= u, the first of the two happens only at u = d (if at all), so all
// other steps are one compare and one select.  A wave holds 64 pivot rows in
// its lanes and reads one a step; unrolled and counted from the first of the
// 64, u is a constant of the instruction (about 16 cycles a step).

// Interchanges u0 .. u0 + 63 (pivot rows in the lanes of pv, highest first; an
// entry equal to its u does nothing) on src; OWN: some lane still follows a
// row of [u0, u0 + 64).
template <bool OWN>
__device__ __forceinline__ void trace64(int &src, int pv, int u0) {
    int r = src - u0;
    const int p = pv - u0;
#pragma unroll
    for (int t = 63; t >= 0; --t) {
        const int q = __builtin_amdgcn_readlane(p, t);
        const int s = r == q ? t : r;
        r = OWN && r == t ? q : s;
    }
    src = r + u0;
}

// A step's interchanges ipiv[j0 .. j0 + cnt) on a strip of columns: every
// workgroup traces the rows that can change (row t < cnt, and the pivot row of
// interchange u where it lies below the block; the same row named twice moves
// the same value twice), then moves them column by column: all loads of a
// column precede its stores.  Tracing takes about 2 us for 256 interchanges;
// by one workgroup ahead of the others, reading the pivots from LDS, it took
// 35 us and a launch.  256 interchanges on the remaining columns, averaged over
// a factorization: n = 5001 74 -> 21 us, n = 8192 90 -> 37 us; 64 at n = 1024:
// 21 -> 10 us.  What is left is the scattered rows: a value of eight bytes
// moves a line of memory.
constexpr int kMaxSwaps = 1024;
constexpr int kSwapCols = 16;   // columns per workgroup

template <typename T, int CPT>
__global__ __launch_bounds__(512) void swap_rows_kernel(T *A, int64_t lda,
                                                        const int32_t *__restrict__ ipiv, int64_t j0,
                                                        int cnt, int64_t nrows, int64_t c_begin,
                                                        int64_t ncols, int64_t skip_begin,
                                                        int64_t skip_len) {
    __shared__ int s_piv[CPT * 256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int nt = blockDim.x;
    const int chunks = (cnt + 63) / 64;
    // relative pivot rows; an entry outside [t, nrows - j0) (possible only in
    // a sequence left by an expired wait) is taken as no interchange, so no
    // row outside the matrix is addressed
    for (int t = tid; t < 64 * chunks; t += nt) {
        const int64_t q = t < cnt ? (int64_t)ipiv[j0 + t] - j0 : t;
        s_piv[t] = (q >= t && q < nrows - j0) ? (int)q : t;
    }
    __syncthreads();
    int dst[CPT], src[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) {
        const int id = tid + nt * e;
        int d = -1;
        if (id < cnt) d = id;
        else if (id < 2 * cnt && s_piv[id - cnt] >= cnt) d = s_piv[id - cnt];
        src[e] = dst[e] = d;
        const int first = id - lane;   // of the wave's candidates
        for (int c = chunks - 1; c >= 0; --c) {
            const int pv = s_piv[64 * c + lane];
            if (first < 64 * c + 64 && first + 64 > 64 * c) trace64<true>(src[e], pv, 64 * c);
            else trace64<false>(src[e], pv, 64 * c);
        }
    }
    constexpr int CB = 8 / CPT;   // columns at a time
    const int64_t q0 = (int64_t)blockIdx.x * kSwapCols;
    const int64_t q1 = q0 + kSwapCols < ncols ? q0 + kSwapCols : ncols;
    const int64_t skip_rel = skip_begin - c_begin;
    for (int64_t qb = q0; qb < q1; qb += CB) {
        T val[CB][CPT];
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const int64_t q = qb + b;
            const int64_t c = c_begin + (q < skip_rel ? q : q + skip_len);
#pragma unroll
            for (int e = 0; e < CPT; ++e)
                if (q < q1 && src[e] != dst[e]) val[b][e] = MXLU_AT(A, j0 + src[e], c, lda);
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const int64_t q = qb + b;
            const int64_t c = c_begin + (q < skip_rel ? q : q + skip_len);
#pragma unroll
            for (int e = 0; e < CPT; ++e)
                if (q < q1 && src[e] != dst[e]) MXLU_AT(A, j0 + dst[e], c, lda) = val[b][e];
        }
    }
}

// ---------------------------------------------------------------------------
// The gather map of the interchanges [0, n): a lane per row, no
// synchronisation.  Row i is not touched by the interchanges after i, so a
// wave starts at its last row.  With `maps`, the state is written out where
// the trace passes a panel boundary: after interchange b nb it is the gather
// map of the interchanges from b nb on, which panel b - 1 needs for its rows
// below (maps: those of b = b0 .. b1 - 1, n ints each).  state: carried from
// the interchanges >= hi; rows before hi have not been touched by those.
// An entry outside [u, n) is taken as no interchange.
// n = 1024 / 5001 / 8192: 13 / 56 / 93 us without maps; with the interchanges
// read as uniform words and two compares and selects a step 43 / 172 / 277.
__global__ __launch_bounds__(64) void perm_trace_kernel(int n, const int32_t *__restrict__ ipiv,
                                                        int lo, int hi, int32_t *__restrict__ state, int nb,
                                                        int b0, int b1, int32_t *__restrict__ maps) {
    const int lane = threadIdx.x;
    const int i0 = 64 * (int)blockIdx.x, i = i0 + lane;
    if (i0 + 64 <= lo) return;
    int src = i < hi || i >= n ? i : state[i];
    int top = min(hi, i0 + 64);   // interchanges [lo, top) remain
    auto pivots = [&](int c) {    // of [64 c, 64 c + 64), outside [lo, top): none
        const int u = 64 * c + lane;
        const int q = u >= lo && u < top ? ipiv[u] : u;
        return q >= u && q < n ? q : u;
    };
    int c = (top - 1) / 64;
    int next = pivots(c);
    // boundaries below top: the highest first
    int b = maps ? min((top - 1) / nb, b1 - 1) : -1;
    for (; c >= 0 && 64 * c + 64 > lo; --c) {
        const int pv = next;
        if (64 * c > lo) next = pivots(c - 1);
        int end = 64;   // of the chunk's interchanges not taken yet
        for (;;) {
            // the rest of the chunk down to a boundary, or all of it
            const bool cut = b >= b0 && b * nb >= 64 * c;
            const int from = cut ? b * nb - 64 * c : 0;
            if (end > from) {
                const int part = lane >= from && lane < end ? pv : 64 * c + lane;
                if (64 * c == i0) trace64<true>(src, part, 64 * c);
                else trace64<false>(src, part, 64 * c);
            }
            if (!cut) break;
            if (i < n) maps[(size_t)(b - b0) * n + i] = src;
            end = from;
            --b;
        }
    }
    if (i < n) state[i] = src;
}

// Deferred interchanges of the columns left of the panels.  No later step
// reads the L columns of a finished panel, so their row interchanges can wait
// until the factorization is done; then each element moves once, through the
// maps above.  A workgroup holds a column's rows below the panel in registers:
// all loads precede the stores, so a column moves in place, and the map is
// read once for kLeftCols columns.  Trace and gather of all panels together:
// n = 1024 (NB = 64) 28 us, n = 5001 100 us, in two launches; six launches per
// panel (compose, map, gather, put back) took 25 to 70 us for each of them.
constexpr int kLeftCols = 4;

template <int NT, int RPT>
__global__ __launch_bounds__(NT) void left_gather_kernel(double *__restrict__ A, int64_t lda, int n,
                                                         int nb, int b0, int first_b,
                                                         const int32_t *__restrict__ maps) {
    const int b = first_b + (int)blockIdx.y;   // panel b - 1, rows from b nb
    const int r0 = b * nb, m = n - r0;
    const int32_t *map = maps + (size_t)(b - b0) * n + r0;
    uint32_t at[RPT / 2];   // rows from r0, two 16-bit numbers a word
    auto row = [&](int e) { return (int)threadIdx.x + NT * e; };
#pragma unroll
    for (int h = 0; h < RPT / 2; ++h) {
        const uint32_t lo = row(2 * h) < m ? (uint32_t)(map[row(2 * h)] - r0) : 0u;
        const uint32_t hi = row(2 * h + 1) < m ? (uint32_t)(map[row(2 * h + 1)] - r0) : 0u;
        at[h] = lo | (hi << 16);
    }
    const int c0 = (int)blockIdx.x * kLeftCols;
    for (int c = c0; c < c0 + kLeftCols && c < nb; ++c) {
        double *col = A + (size_t)r0 + (size_t)(r0 - nb + c) * (size_t)lda;
        double val[RPT];
#pragma unroll
        for (int e = 0; e < RPT; ++e)
            if (row(e) < m) val[e] = col[e & 1 ? at[e / 2] >> 16 : at[e / 2] & 0xffffu];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < RPT; ++e)
            if (row(e) < m) col[row(e)] = val[e];
    }
}
constexpr int64_t kLeftRows = 1024 * 32;   // rows below a panel that it can hold (16-bit numbers)

// Taller ones through T (rows x cols, leading dimension rows): T <- the
// gathered rows, then back.
__global__ void gather_panel_rows_kernel(const double *__restrict__ A, int64_t lda, int64_t r0,
                                         int64_t rows, int64_t c0, const int32_t *__restrict__ q,
                                         double *__restrict__ T) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t c = blockIdx.y;
    if (i < rows) T[i + c * rows] = MXLU_AT(A, q[r0 + i], c0 + c, lda);
}

// A[r0 + i, c0 + c] <- T
__global__ void put_panel_rows_kernel(const double *__restrict__ T, int64_t rows, double *__restrict__ A,
                                int64_t lda, int64_t r0, int64_t c0) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t c = blockIdx.y;
    if (i < rows) MXLU_AT(A, r0 + i, c0 + c, lda) = T[i + c * rows];
}

int trace(int64_t n, const int32_t *ipiv, int64_t lo, int64_t hi, int32_t *state, int64_t nb,
          int64_t b0, int64_t b1, int32_t *maps, hipStream_t s) {
    hipLaunchKernelGGL(perm_trace_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, (int)n,
                       ipiv, (int)lo, (int)hi, state, (int)nb, (int)b0, (int)b1, maps);
    MXLU_LAUNCH_CHECK();
    return 0;
}

}  // namespace

namespace mxlu {

template <typename T>
int swap_rows(T *A, int64_t lda, int64_t nrows, const int32_t *ipiv, int64_t j0, int cnt,
              int64_t c_begin, int64_t ncols, int64_t skip_begin, int64_t skip_len, hipStream_t s) {
    if (cnt <= 0 || ncols <= 0) return 0;
    if (cnt > kMaxSwaps || nrows - j0 > INT_MAX || ncols > (int64_t)INT_MAX * kSwapCols) {
        set_error_msg("laswp: too many interchanges, rows or columns");
        return MXLU_E_NOMEM;
    }
    const dim3 grid((unsigned)((ncols + kSwapCols - 1) / kSwapCols));
    const dim3 block((unsigned)std::min(512, (2 * cnt + 63) / 64 * 64));
    if (cnt <= 256)
        hipLaunchKernelGGL((swap_rows_kernel<T, 1>), grid, block, 0, s, A, lda, ipiv, j0, cnt, nrows,
                           c_begin, ncols, skip_begin, skip_len);
    else if (cnt <= 512)
        hipLaunchKernelGGL((swap_rows_kernel<T, 2>), grid, block, 0, s, A, lda, ipiv, j0, cnt, nrows,
                           c_begin, ncols, skip_begin, skip_len);
    else
        hipLaunchKernelGGL((swap_rows_kernel<T, 4>), grid, block, 0, s, A, lda, ipiv, j0, cnt, nrows,
                           c_begin, ncols, skip_begin, skip_len);
    MXLU_LAUNCH_CHECK();
    return 0;
}
template int swap_rows<double>(double *, int64_t, int64_t, const int32_t *, int64_t, int, int64_t,
                               int64_t, int64_t, int64_t, hipStream_t);
template int swap_rows<float>(float *, int64_t, int64_t, const int32_t *, int64_t, int, int64_t,
                              int64_t, int64_t, int64_t, hipStream_t);
template int swap_rows<uint16_t>(uint16_t *, int64_t, int64_t, const int32_t *, int64_t, int, int64_t,
                                 int64_t, int64_t, int64_t, hipStream_t);

int perm_from_ipiv(int64_t n, const int32_t *ipiv, int32_t *perm, hipStream_t s) {
    if (n <= 0) return 0;
    return trace(n, ipiv, 0, n, perm, 1, 0, 0, nullptr, s);
}

// panels whose maps are held at once: 64 MB, one at least
static int64_t left_batch(int64_t n, int64_t nb) {
    return std::max<int64_t>(1, std::min<int64_t>((n + nb - 1) / nb - 1, ((int64_t)1 << 24) / n));
}

int64_t left_swap_map_ints(int64_t n, int64_t nb) { return n > nb ? (left_batch(n, nb) + 1) * n : 0; }
int64_t left_swap_rows(int64_t n, int64_t nb) { return n - nb > kLeftRows ? n - nb : 0; }

int laswp_left_deferred_f64(double *A, int64_t lda, int64_t n, int64_t nb, const int32_t *ipiv,
                            int32_t *maps, double *T, hipStream_t s) {
    const int64_t K = (n + nb - 1) / nb, batch = left_batch(n, nb);
    if (K < 2) return 0;
    int32_t *state = maps + batch * n;
    for (int64_t b1 = K; b1 > 1; b1 -= batch) {   // boundaries b0 .. b1 - 1, last ones first
        const int64_t b0 = std::max<int64_t>(1, b1 - batch);
        MXLU_TRY(trace(n, ipiv, b0 * nb, std::min(n, b1 * nb), state, nb, b0, b1, maps, s));
        int64_t b = b0;
        for (; b < b1 && n - b * nb > kLeftRows; ++b) {
            const int64_t rows = n - b * nb;
            const dim3 grid((unsigned)((rows + 255) / 256), (unsigned)nb);
            const int32_t *map = maps + (b - b0) * n;
            hipLaunchKernelGGL(gather_panel_rows_kernel, grid, dim3(256), 0, s, A, lda, b * nb, rows,
                               (b - 1) * nb, map, T);
            MXLU_LAUNCH_CHECK();
            hipLaunchKernelGGL(put_panel_rows_kernel, grid, dim3(256), 0, s, T, rows, A, lda, b * nb,
                               (b - 1) * nb);
            MXLU_LAUNCH_CHECK();
        }
        for (; b < b1; b += 65535) {   // (a grid's y is at most 65535)
            const int64_t m = n - b * nb;
            const dim3 grid((unsigned)((nb + kLeftCols - 1) / kLeftCols),
                            (unsigned)std::min<int64_t>(65535, b1 - b));
            // the smallest workgroup that holds the tallest panel's rows
            if (m <= 2048)
                hipLaunchKernelGGL((left_gather_kernel<256, 8>), grid, dim3(256), 0, s, A, lda, (int)n,
                                   (int)nb, (int)b0, (int)b, maps);
            else if (m <= 8192)
                hipLaunchKernelGGL((left_gather_kernel<512, 16>), grid, dim3(512), 0, s, A, lda, (int)n,
                                   (int)nb, (int)b0, (int)b, maps);
            else
                hipLaunchKernelGGL((left_gather_kernel<1024, 32>), grid, dim3(1024), 0, s, A, lda,
                                   (int)n, (int)nb, (int)b0, (int)b, maps);
            MXLU_LAUNCH_CHECK();
        }
    }
    return 0;
}

}  // namespace mxlu
